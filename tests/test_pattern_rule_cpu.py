"""Which plain products read row patterns, on the CPU (the dispatch rule built
as host code).  Block widths and sizes that were measured slower from patterns
than from codes must stay on codes: binary64 rows of odd width (m = 9 at 19,683
rows 9 % slower, m = 13 at 294,912 rows 9 %) and rows of five lanes on small
matrices.  Those measured faster must keep patterns."""
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

    def ask(size, m, n):
        r = subprocess.run([exe, str(size), str(m), str(n)], capture_output=True, text=True, check=True)
        return r.stdout == "1\n"
    return ask


@pytest.mark.parametrize("size,m,n", [(8, 5, 19683), (8, 5, 49152), (8, 5, 110592), (8, 7, 19683), (8, 7, 27000),
                                      (8, 9, 19683), (8, 9, 294912), (8, 9, 389851), (8, 13, 49152), (8, 13, 294912), (8, 13, 819200),
                                      (8, 15, 110592), (8, 15, 294912), (8, 15, 819200), (8, 10, 49152), (8, 10, 110592),
                                      (4, 5, 110592), (4, 10, 110592)])
def test_slower_from_patterns(reads_patterns, size, m, n):
    assert not reads_patterns(size, m, n)


@pytest.mark.parametrize("size,m,n", [(8, 1, 19683), (8, 2, 27000), (8, 1, 12582912), (8, 4, 524288), (8, 5, 389851),
                                      (8, 7, 938091), (8, 9, 524288), (8, 10, 184320), (8, 16, 19683), (8, 16, 110592),
                                      (4, 1, 65536), (4, 4, 27000), (4, 5, 184320), (4, 8, 524288), (4, 11, 49152),
                                      (4, 13, 27000), (4, 16, 938091)])
def test_faster_from_patterns(reads_patterns, size, m, n):
    assert reads_patterns(size, m, n)
