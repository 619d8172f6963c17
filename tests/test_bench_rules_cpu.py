"""The benchmark's offline accounting, without a device: which kernels a trace
names and how many matrix bytes it credits them with."""
import bench
from workloads import grids

PAT = "void mrhs::k_gspmv_pat<double, 1, mrhs::OpStore<double, 1> >(mrhs::CsrView<double>, int)"
STAGED = "void mrhs::k_gspmv<double, 16, mrhs::OpSpmv1<double, 16> >(mrhs::CsrView<double>, int)"


def test_bytes_of_pattern_kernels():
    """A product that read row patterns is credited with 2 bytes per row, not
    with the codes it did not read."""
    A = grids.dirichlet7(10)
    codes = 4 * (A.n + 1) + 2 * A.nnz
    assert bench.kernel_class(PAT) == "gspmv/f64/m1" and bench.kernel_class(STAGED) == "spmv_sigma/f64/m16"
    assert bench.summary_mat(A, "gspmv", 8, PAT) == 2 * A.n
    assert bench.summary_mat(A, "spmv_sigma", 8, STAGED) == codes
    assert bench.summary_mat(A, "xr_update", 8, STAGED) is None
    byt = bench.kernel_bytes("gspmv", A.n, A.nnz, 1, 8, bench.summary_mat(A, "gspmv", 8, PAT))
    assert byt == 2 * A.n + 2 * 8 * A.n


def test_dominant_kernel_takes_its_own_matrix_bytes():
    n, nnz, m = 1000, 6400, 16
    trace = {"spmv_omega/f64/m16/g512": {"launches": 4, "seen": 4, "total_ms": 4.0},
             "xr_update/f64/m16/g512": {"launches": 4, "seen": 4, "total_ms": 1.0}}
    d = bench.dominant_kernel(trace, n, nnz, {("spmv_sigma", 8): 16800, ("spmv_omega", 8): 2000})
    assert d["bytes_per_launch"] == 2000 + 3 * 8 * m * n


def test_every_kernel_has_a_name():
    for symbol, cls in (
            ("void mrhs::k_cols<mrhs::OpColDots>(mrhs::ColBatch, int)", "gcr_dots/f64/m1"),
            ("void mrhs::k_cols<mrhs::OpColUpdate>(mrhs::ColBatch, int)", "gcr_update/f64/m1"),
            ("void mrhs::k_gspmv_split<float, 8, mrhs::OpVcRes<float, 8> >(mrhs::CsrView<float>, int)", "vc_resid/f32/m8"),
            ("void mrhs::k_stream<double, 16, mrhs::OpXR<double, 16> >(int)", "xr_update/f64/m16"),
            ("void mrhs::k_gspmv_march<double, 8, mrhs::OpStore<double, 8> >(int)", "gspmv/f64/m8")):
        assert bench.kernel_class(symbol) == cls
    assert bench.kernel_class("mrhs::k_ctl_reset(mrhs::Ctl*)") == "mrhs::k_ctl_reset"
