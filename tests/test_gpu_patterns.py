"""GPU parity of the row-pattern form of a matrix (csr_create).

Where the rows of a matrix with 16-bit codes repeat, products read one pattern
number per row and a table of patterns.  They sum the same values in the same
order as from codes (MRHS_CSR_PATTERN=0) and from the plain arrays
(MRHS_CSR_DICT=0), and every form adds the partial dot products in one order,
so products and solves must agree bit for bit.  Covered: grids whose lines are
shorter and longer than a wave's rows, sizes that leave ragged tiles and waves,
rows whose near entries are missing, out of the stencil's order or repeated,
empty rows, rows longer than a batch, both value precisions, every block width,
non-finite block values, and matrices on both sides of the sizes where products
change form.
"""
import os

import numpy as np
import pytest

from workloads import grids, rng
from workloads.grids import CSRMatrix

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1711_10622_amd as p
    p.load(build_if_missing=False)
    return torch, p


def make(p, A, **env):
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        return p.CsrMatrix.from_csr(A)
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.update({k: v})


def from_rows(n, row_of):
    """Row i holds the (offset, value) pairs of row_of(i) in that order."""
    rp, ci, va = [0], [], []
    for i in range(n):
        for o, v in row_of(i):
            ci.append(i + o)
            va.append(v)
        rp.append(len(ci))
    return CSRMatrix(n, np.array(rp, np.int32), np.array(ci, np.int32), np.array(va, np.float64))


def inside(n, i, entries):
    return [(o, v) for o, v in entries if 0 <= i + o < n]


def shuffled(n):
    """Entries out of column order and a repeated one (no stencil shape), every
    fifth row empty, every seventh without its diagonal."""
    def row(i):
        if i % 5 == 4:
            return []
        e = [(40, -1.0), (0, 6.0), (-1, -1.5), (1, -0.5), (0, 0.25), (-40, -2.0)]
        return inside(n, i, [x for x in e if not (i % 7 == 0 and x[0] == 0)])
    return from_rows(n, row)


def band(n, half):
    return from_rows(n, lambda i: inside(n, i, [(o, 40.0 if o == 0 else -1.0 - 0.5 * (o % 2))
                                                for o in range(-half, half + 1)]))


CASES = {
    "chan131x9x7": lambda: grids.channel7(131, 9, 7, beta=2.0),
    "chan24x40x33": lambda: grids.channel7(24, 40, 33, beta=2.0),
    "dir33x32x31": lambda: grids.dirichlet7(33, 32, 31),
    "dir5x300x20": lambda: grids.dirichlet7(5, 300, 20),
    "dir26x26x26": lambda: grids.dirichlet7(26),  # 17,576 rows: past the small-matrix line
    "shuffled": lambda: shuffled(20011),
    "band9": lambda: band(16411, 9),
}


def cuda(torch, X):
    return torch.from_numpy(np.ascontiguousarray(X)).cuda()


@pytest.mark.parametrize("name", list(CASES))
def test_products_bitwise(env, name):
    torch, p = env
    A = CASES[name]()
    M = make(p, A)
    forms = [make(p, A, MRHS_CSR_PATTERN="0"), make(p, A, MRHS_CSR_DICT="0")]
    for m in range(1, 17):
        X = rng.rhs_block(A.n, m, 500 + m)
        X[3 % A.n, 0] = np.inf
        X[A.n // 2, m - 1] = np.nan
        for Xt in (X, X.astype(np.float32)):
            Y = M.gspmv(cuda(torch, Xt)).cpu().numpy()
            for F in forms:
                assert np.array_equal(Y, F.gspmv(cuda(torch, Xt)).cpu().numpy(), equal_nan=True), (m, Xt.dtype)
    for h in (M, *forms):
        h.close()


@pytest.mark.parametrize("name,m,mixed", [
    ("chan131x9x7", 1, False), ("chan131x9x7", 8, False), ("dir5x300x20", 4, False),
    ("dir5x300x20", 16, False), ("dir26x26x26", 3, False), ("dir26x26x26", 12, False), ("chan24x40x33", 8, True),
    ("dir33x32x31", 16, True),
])
def test_solves_bitwise(env, name, m, mixed):
    """Sigma, omega, update and residual passes: 30 iterations."""
    torch, p = env
    A = CASES[name]()
    B = rng.rhs_block(A.n, m, 600 + m, mean_zero=bool(A.nullspace_const))
    out = []
    for kw in ({}, {"MRHS_CSR_PATTERN": "0"}, {"MRHS_CSR_DICT": "0"}):
        M = make(p, A, **kw)
        X, infos, st = M.solve(cuda(torch, B), tol=1e-14, maxit=30, mixed=mixed)
        out.append((X.cpu().numpy(), [(i["iters"], i["relres"]) for i in infos], st))
        M.close()
    for o in out[1:]:
        assert o[1] == out[0][1] and o[2] == out[0][2]
        assert np.array_equal(o[0], out[0][0])


def test_large_matrix_bitwise(env):
    """Past 2^21 rows narrow rows read patterns, the rest codes; one plane of
    50 x 41 rows is not a whole number of tiles."""
    torch, p = env
    A = grids.dirichlet7(50, 41, 1025)
    assert A.n > 1 << 21
    M, F = make(p, A), make(p, A, MRHS_CSR_PATTERN="0")
    for m in (1, 2, 5, 8, 16):
        X = rng.rhs_block(A.n, m, 700 + m)
        for Xt in (X, X.astype(np.float32)):
            assert np.array_equal(M.gspmv(cuda(torch, Xt)).cpu().numpy(), F.gspmv(cuda(torch, Xt)).cpu().numpy()), m
    for m in (1, 7, 16):
        B = cuda(torch, rng.rhs_block(A.n, m, 800 + m))
        X = [h.solve(B, tol=1e-30, maxit=6)[0].cpu().numpy() for h in (M, F)]
        assert np.array_equal(X[0], X[1]), m
    M.close()
    F.close()
