"""What row patterns cost in device memory: a pattern number per row and the
tables that some product reads.  Plain products read A's entries; the two-block
omega pass, past 2^21 rows alone, the entries and stencils of A D^-1."""
import os

import pytest

from workloads import grids

pytestmark = pytest.mark.gpu

PATTERNS, ENTRIES = 27, 8  # a cell layer of each kind; whole batches of the seven entries
ENTRY = {8: 16, 4: 8}
STENCIL = {8: 80, 4: 48}


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1711_10622_amd as p
    p.load(build_if_missing=False)
    return p


def bytes_of(p, A, pattern):
    old = os.environ.get("MRHS_CSR_PATTERN")
    os.environ["MRHS_CSR_PATTERN"] = pattern
    try:
        M = p.CsrMatrix.from_csr(A)
    finally:
        os.environ.pop("MRHS_CSR_PATTERN") if old is None else os.environ.update({"MRHS_CSR_PATTERN": old})
    b = M.device_bytes()
    M.close()
    return b


@pytest.mark.parametrize("shape", [(33, 32, 31), (64, 64, 64), (131, 127, 127)])
def test_bytes_of_patterns(env, shape):
    A = grids.dirichlet7(*shape)
    entries = PATTERNS * ENTRIES * (ENTRY[8] + ENTRY[4])
    tables = entries
    if A.n > 1 << 21:
        tables += entries + PATTERNS * (STENCIL[8] + STENCIL[4])
    assert bytes_of(env, A, "1") - bytes_of(env, A, "0") == 2 * A.n + 4 * PATTERNS + tables
