"""GPU parity of the row-pattern products at the sizes and widths that run them.

Every matrix here is shown to hold patterns (its handle is larger than the one
made with MRHS_CSR_PATTERN=0) and reads them in every product that has a kernel
for them (MRHS_CSR_PATTERN=2), also where codes would be faster; products and
solves must give the bits of the coded and plain forms.  Past 2^21 rows the
omega pass of both precisions reads patterns through gspmv_near_pat: waves whose
rows are one whole stencil, one partial stencil (at a wall), several patterns
(line ends) and no stencil at all.
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


def forms(p, A):
    """The handle under test and the ones it must agree with."""
    M, F, P = (make(p, A, MRHS_CSR_PATTERN="2"), make(p, A, MRHS_CSR_PATTERN="0"), make(p, A, MRHS_CSR_DICT="0"))
    assert M.device_bytes() > F.device_bytes()  # patterns are there
    if A.n <= 1 << 21:
        assert all(M.product_bytes(m, dt) < F.product_bytes(m, dt) for dt in ("f64", "f32") for m in range(1, 17)
                   if dt == "f32" or m not in (13, 15))
    else:
        assert all(M.product_bytes(m, dt, "spmv_omega") < F.product_bytes(m, dt, "spmv_omega")
                   for dt in ("f64", "f32") for m in range(1, 17))
    return M, F, P


def banded(n, offsets, values, drop=()):
    """Row i holds (i + offsets[k], values[k]) in that order where the column
    exists; drop: (modulus, remainder, k) leaves entry k out of such rows."""
    offs = np.asarray(offsets)
    cols = np.arange(n, dtype=np.int64)[:, None] + offs[None, :]
    ok = (cols >= 0) & (cols < n)
    for mod, rem, k in drop:
        ok[np.arange(n) % mod == rem, k] = False
    vals = np.broadcast_to(np.asarray(values, np.float64), cols.shape)
    rp = np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32)
    return CSRMatrix(n, rp, cols[ok].astype(np.int32), np.ascontiguousarray(vals[ok]))


def cuda(torch, X):
    return torch.from_numpy(np.ascontiguousarray(X)).cuda()


# lines longer and much shorter than a wave's rows, ragged tiles, rows out of the
# stencil's order with repeated and missing entries, rows of two and a half
# gather batches
CASES = {
    "chan131x67x61": lambda: grids.channel7(131, 67, 61, beta=2.0),
    "dir5x331x331": lambda: grids.dirichlet7(5, 331, 331),
    "shuffled": lambda: banded(530011, (40, 0, -1, 1, 0, -40), (-1.0, 6.0, -1.5, -0.5, 0.25, -2.0),
                               ((7, 0, 1), (5, 4, 5))),
    "band19": lambda: banded(528391, range(-9, 10), [40.0 if o == 0 else -1.0 - 0.5 * (o % 2) for o in range(-9, 10)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_products_bitwise(env, name):
    torch, p = env
    A = CASES[name]()
    M, *others = forms(p, A)
    for m in range(1, 17):
        X = rng.rhs_block(A.n, m, 1500 + m)
        X[3, 0] = np.inf
        X[A.n // 2, m - 1] = np.nan
        for Xt in (X, X.astype(np.float32)):
            Y = M.gspmv(cuda(torch, Xt))
            for F in others:
                assert torch.equal(Y.view(torch.uint8), F.gspmv(cuda(torch, Xt)).view(torch.uint8)), (m, Xt.dtype)
    for h in (M, *others):
        h.close()


@pytest.mark.parametrize("scale", [1.0, 3e-41, 1e-45, 1e-310])
def test_rounded_values_bitwise(env, scale):
    """The tables of the binary32 products are rounded on the host, the plain
    binary32 arrays on the device: subnormal and vanishing values too."""
    torch, p = env
    A = banded(20011, (-40, -1, 0, 1, 40), (-1.0 / 3, -1.5, 6.0 / 7, -0.7, -2.1))
    A = CSRMatrix(A.n, A.row_ptr, A.col, A.val * scale)
    M, *others = forms(p, A)
    for m in (1, 4, 7):
        X = rng.rhs_block(A.n, m, 1600 + m) * 1e6
        for Xt in (X, X.astype(np.float32)):
            Y = M.gspmv(cuda(torch, Xt))
            for F in others:
                assert torch.equal(Y, F.gspmv(cuda(torch, Xt))), (m, Xt.dtype)
    for h in (M, *others):
        h.close()


LARGE = {
    "chan130x97x170": lambda: grids.channel7(130, 97, 170, beta=2.0),  # lines of two waves and two rows
    "dir200x103x103": lambda: grids.dirichlet7(200, 103, 103),
    # no stencil: the diagonal is not between its neighbours
    "order": lambda: banded((1 << 21) + 777, (300, 0, -1, 1, -300), (-1.0, 7.0, -1.5, -0.5, -2.0)),
    # a stencil of two distant entries whose rows drop one neighbour in turn
    "partial": lambda: banded((1 << 21) + 777, (-300, -1, 0, 1, 300), (-1.0, -1.5, 7.0, -0.5, -2.0),
                              ((4096, 0, 1), (512, 3, 3))),
}


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("name", list(LARGE))
def test_large_solves_bitwise(env, name, mixed):
    torch, p = env
    A = LARGE[name]()
    assert A.n > 1 << 21
    M, F, P = forms(p, A)
    for m in (1, 4, 7, 16):
        B = cuda(torch, rng.rhs_block(A.n, m, 1700 + m, mean_zero=bool(A.nullspace_const)))
        out = []
        for h in (M, F, P):
            X, infos, st = h.solve(B, tol=1e-30, maxit=6, mixed=mixed)
            out.append((X, [(i["iters"], i["relres"]) for i in infos], st))
        for o in out[1:]:
            assert o[1:] == out[0][1:], m
            assert torch.equal(o[0], out[0][0]), m
    for h in (M, F, P):
        h.close()
