"""GPU parity of the forms in which multigrid levels are read.

The tiled products of a level read codes (MRHS_CSR_DICT=0: the plain arrays)
and sum the same values in the same order, so V-cycles agree bit for bit
between the forms where every product runs tiled, and to rounding where the
short-chain product orders a row's sum its own way.  Levels hold no row
patterns (MRHS_CSR_PATTERN), whatever the matrix's own products read.
"""
import os

import numpy as np
import pytest

from workloads import grids, rng

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1711_10622_amd as p
    p.load(build_if_missing=False)
    return torch, p


def hierarchy(p, A, **env):
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        M = p.CsrMatrix.from_csr(A)
        return M, p.AmgHierarchy(M)
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.update({k: v})


def vcycles(torch, H, B):
    """One V-cycle in binary64 and one solve of two iterations with binary32
    V-cycles."""
    Bd = torch.from_numpy(B).cuda()
    Y = H.vcycle(Bd).cpu().numpy()
    X, infos, _ = H.solve(Bd, tol=1e-30, maxit=2, mixed=True)
    return Y, X.cpu().numpy(), [i["relres"] for i in infos]


@pytest.mark.parametrize("name,m", [("chan", 1), ("chan", 7), ("chan", 16), ("dir", 5), ("dir", 8)])
def test_levels_read_codes(env, name, m):
    """A finest level past 131,072 rows, where the matrix has patterns: its
    hierarchy holds the same bytes and gives the same bits without them."""
    torch, p = env
    A = grids.channel7(72, 48, 40, beta=2.0) if name == "chan" else grids.dirichlet7(53, 51, 50)
    assert A.n > 131072
    B = rng.rhs_block(A.n, m, 900 + m, mean_zero=bool(A.nullspace_const))
    (M, H), (N, F) = hierarchy(p, A), hierarchy(p, A, MRHS_CSR_PATTERN="0")
    assert M.device_bytes() > N.device_bytes()  # the matrix itself has patterns
    assert H.device_bytes == F.device_bytes
    for a, b in zip(vcycles(torch, H, B), vcycles(torch, F, B)):
        assert np.array_equal(a, b)
    for h in (H, F, M, N):
        h.close()


def test_short_rows_of_small_levels_are_coded(env):
    """Plane of 300 x 300: the second level, 45,000 rows of nine entries, is
    coded beside the first (2 bytes per entry of A_l and of A_l D_l1^-1), and
    widths that run tiled there (3, 5, 7, 9) give the plain arrays' bits."""
    torch, p = env
    A = grids.dirichlet7(300, 300, 1)
    (M, H), (N, F) = hierarchy(p, A), hierarchy(p, A, MRHS_CSR_DICT="0")
    n1, nnz1 = H.level(1)[:2]
    assert n1 < 131072 and nnz1 < 12 * n1
    assert H.device_bytes - F.device_bytes >= 4 * (A.nnz + nnz1)
    for m in (3, 5, 7, 9):
        B = rng.rhs_block(A.n, m, 950 + m)
        for a, b in zip(vcycles(torch, H, B), vcycles(torch, F, B)):
            assert np.array_equal(a, b)
    for h in (H, F, M, N):
        h.close()
