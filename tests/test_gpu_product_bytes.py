"""The bytes a product reads from the matrix arrays, as the library reports them
for each form: row patterns where the product reads them, else what
csr_stream_bytes says, whatever the handle also holds."""
import os

import pytest

from workloads import grids, rng

pytestmark = pytest.mark.gpu

OPS = ("gspmv", "spmv_sigma", "spmv_omega")


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1711_10622_amd as p
    p.load(build_if_missing=False)
    return p


def make(p, A, reorder=False, **env):
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        return p.CsrMatrix.from_csr(A, reorder=reorder)
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.update({k: v})


def table(dtype, omega=False):
    """27 kinds of row of a Dirichlet grid, eight entries' room each."""
    size = 8 if dtype == "f64" else 4
    return 27 * (4 + 8 * 2 * size + (80 if size == 8 else 48) * omega)


# widths whose products read patterns: lines of 64 rows (runs of 21), and past
# 2^21 rows lines of 131 (runs of 43)
READ = {
    (64, "f64", "gspmv"): {1, 2, 4, 6, 8, 10, 12, 14, 16}, (64, "f32", "gspmv"): set(range(1, 17)),
    (131, "f64", "gspmv"): {1, 2}, (131, "f32", "gspmv"): {1, 2, 3, 4},
    (131, "f64", "spmv_omega"): set(range(1, 17)), (131, "f32", "spmv_omega"): set(range(1, 17)),
}


@pytest.mark.parametrize("shape", [(64, 64, 64), (131, 127, 127)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_bytes_follow_the_form(env, shape, dtype):
    A = grids.dirichlet7(*shape)
    M, F = make(env, A), make(env, A, MRHS_CSR_PATTERN="0")
    assert M.stream_bytes(dtype, True) == 4 * (A.n + 1) + 2 * A.nnz
    for m in range(1, 17):
        for op in OPS:
            codes = M.stream_bytes(dtype, op != "gspmv")
            assert F.product_bytes(m, dtype, op) == codes
            reads = m in READ.get((shape[0], dtype, op), ())
            want = 2 * A.n + table(dtype, op == "spmv_omega") if reads else codes
            assert M.product_bytes(m, dtype, op) == want, (m, op)
    M.close()
    F.close()


def test_other_forms(env):
    A = grids.permute_symmetric(grids.dirichlet7(26), rng.permutation(26 ** 3, 3))
    M = make(env, A)
    assert M.product_bytes(4) == M.stream_bytes() == 4 * (A.n + 1) + 4 * A.nnz
    R = make(env, A, reorder=True)
    assert R.product_bytes(4) == 4 * (A.n + 1) + 12 * A.nnz  # the caller's arrays
    assert R.product_bytes(4, "f64", "spmv_sigma") == R.stream_bytes("f64", True)
    for bad in (dict(m=0), dict(m=17)):
        with pytest.raises(Exception):
            M.product_bytes(**bad)
    M.close()
    R.close()
