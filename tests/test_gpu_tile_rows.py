"""Reducing kernels on small matrices, where tiles hold fewer passes.

A kernel with a grid reduction takes tiles of as many passes as leave each
compute unit one (up to 256 rows), so the passes per tile change at multiples of
compute units times the rows of a pass.  Short solves at sizes just below, at
and past such lines, with ragged last tiles, run the sigma, omega, update and
residual passes over all three matrix forms.

Tolerance against the oracle: rounding moves a dot product of n values and the
random shadow residual by at most about n u sqrt(n) = 2e-9 at n = 66,000; a row
left out or taken twice moves one by 1 / n = 1.5e-5.  1e-8 lies between.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1711_10622_amd._lib import SHADOW_SEED
from workloads import grids, rng
from workloads.grids import CSRMatrix

pytestmark = pytest.mark.gpu

ITERS = 2


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1711_10622_amd as p
    p.load(build_if_missing=False)
    return torch, p


def pass_rows(m):
    """Rows of one pass of a workgroup in binary64 and the passes of a full tile."""
    vw = 2 if m % 2 == 0 else 1
    g = m // vw
    pow2 = 1 << (g - 1).bit_length()
    lanes = g if (vw == 1 or g == 5) and 64 // g > 64 // pow2 else pow2
    rows = 4 * (64 // lanes)
    return rows, max(1, 256 // rows)


def band(n):
    offs = np.array([-40, -1, 0, 1, 40])
    cols = np.arange(n)[:, None] + offs[None, :]
    ok = (cols >= 0) & (cols < n)
    vals = np.broadcast_to(np.array([-1.0, -1.5, 7.0, -0.5, -2.0]), cols.shape).copy()
    vals[:, 2] += np.arange(n) % 3
    rp = np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32)
    return CSRMatrix(n, rp, cols[ok].astype(np.int32), np.ascontiguousarray(vals[ok]))


def solve(torch, p, A, B, plain=False, **kw):
    old = os.environ.get("MRHS_CSR_DICT")
    os.environ["MRHS_CSR_DICT"] = "0" if plain else "1"
    try:
        M = p.CsrMatrix.from_csr(A)
    finally:
        os.environ.pop("MRHS_CSR_DICT") if old is None else os.environ.update({"MRHS_CSR_DICT": old})
    X, infos, st = M.solve(torch.from_numpy(B).cuda(), **kw)
    per = (M.stream_bytes("f64", True) - 4 * (A.n + 1)) // len(A.col)
    M.close()
    return X.cpu().numpy(), [(i["iters"], i["relres"]) for i in infos], per


@pytest.mark.parametrize("m", [3, 4, 5, 7, 8, 16])
def test_solves_where_tiles_change(env, m):
    torch, p = env
    rows, full = pass_rows(m)
    unit = torch.cuda.get_device_properties(0).multi_processor_count * rows
    for n in sorted({k * unit + d for k in (1, 2, full) for d in (-1, 0, 1, rows // 2)}):
        A = band(n)
        R = grids.permute_symmetric(A, rng.permutation(n, 17))
        B = rng.rhs_block(n, m, 1800 + m)
        for C, entry in ((A, 2), (R, 4)):  # 16-bit codes, column codes
            X, infos, per = solve(torch, p, C, B, tol=1e-14, maxit=ITERS)
            Xp, infosp, plain = solve(torch, p, C, B, plain=True, tol=1e-14, maxit=ITERS)
            assert (per, plain) == (entry, 12)
            assert np.array_equal(X, Xp) and infos == infosp, n
            Xo, io, _ = oracle.bicgstab(C, B, tol=1e-14, maxit=ITERS, shadow_seed=SHADOW_SEED, threads=4)
            for l in range(m):
                assert infos[l][0] == io[l]["iters"] == ITERS
                assert np.linalg.norm(X[:, l] - Xo[:, l]) <= 1e-8 * np.linalg.norm(Xo[:, l]), (n, l)
                assert abs(infos[l][1] - io[l]["relres"]) <= 1e-8 * io[l]["relres"], (n, l)


@pytest.mark.parametrize("m", [7, 16])
def test_mixed_solves_where_tiles_change(env, m):
    torch, p = env
    rows, full = pass_rows(m)
    unit = torch.cuda.get_device_properties(0).multi_processor_count * rows
    for n in (unit - 1, 2 * unit + 1, full * unit):
        A = band(n)
        B = rng.rhs_block(n, m, 1900 + m)
        X, infos, _ = solve(torch, p, A, B, tol=1e-10, mixed=True)
        Xp, infosp, _ = solve(torch, p, A, B, plain=True, tol=1e-10, mixed=True)
        assert np.array_equal(X, Xp) and infos == infosp, n
        R = B - oracle.gspmv_dot2(A, X)
        assert np.all(np.linalg.norm(R, axis=0) <= 1e-10 * np.linalg.norm(B, axis=0)), n
