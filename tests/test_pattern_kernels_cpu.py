"""Which row-pattern kernels the library holds, on the CPU: one for every
product that dispatch can send to it (plain products, the columns' product of
refinement, the two-block omega pass) and none for any other.  A kernel that
nothing can launch is time to compile and bytes to load."""
import re
import shutil
import subprocess

import pytest

from paper_1711_10622_amd import _lib, build


@pytest.fixture(scope="module")
def kernels():
    nm = shutil.which("nm") or shutil.which("llvm-nm")
    if nm is None:
        pytest.skip("nm not available")
    _lib.load(build_if_missing=True)
    text = subprocess.run([nm, "-C", build.LIB], capture_output=True, text=True, check=True).stdout
    return set(re.findall(r"k_gspmv_pat<(double|float), (\d+), mrhs::(\w+)<", text))


def test_only_reachable_kernels(kernels):
    assert {op for _, _, op in kernels} == {"OpStore", "OpColsStore", "OpSpmv2"}


def test_every_reachable_kernel(kernels):
    widths = {str(m) for m in range(1, 17)}
    for op in ("OpStore", "OpSpmv2"):
        for t in ("double", "float"):
            have = {m for tt, m, o in kernels if (tt, o) == (t, op)}
            never = {"13", "15"} if (t, op) == ("double", "OpStore") else set()  # slower at every size
            assert have == widths - never, (op, t)
