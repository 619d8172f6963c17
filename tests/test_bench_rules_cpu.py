"""The benchmark's offline accounting, without a device: which kernels a trace
names and how many matrix bytes it credits them with."""
import json

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
    anonymous = "void mrhs::k_gspmv_split<double, 1, mrhs::(anonymous namespace)::OpVcSmooth<double, 1> >(int)"
    assert bench.kernel_class(anonymous) == "vc_smooth/f64/m1"
    assert bench.kernel_class("mrhs::(anonymous namespace)::k_to_user(double*)") == "mrhs::k_to_user"


RESULT = {"metric": bench.METRIC, "value": 0.6345, "unit": "s/RHS", "n_gpus": 1, "steps": 20, "warmup": 5,
          "ms_per_step": 10151.2, "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
          "data": "synthetic", "config": {"workload": "w" * 300, "n": 12582912, "m": 16},
          "cpu_baseline": {"value": 33.1, "sample": "s" * 400}}


def sweep(ms):
    return {f"{dt}/m{m}": {"us_median": 123.456789, "us_p10": 120.1, "us_p90": 130.2, "GBps": 4321.987,
                           "frac_hbm_peak": 0.5402} for dt in ("f64", "f32") for m in ms}


def test_line_can_be_read_whole():
    """All legs of a full run: one line that a reader of the last 8000
    characters still finds, with the result's own fields as they were."""
    extra = {"iters": list(range(1000, 1016)), "iters_max": 1974, "gspmv_chan256": sweep(range(1, 17)),
             "gspmv_cube192": {"relabelled": sweep((8, 16)), "rcm": sweep((8, 16))},
             "amg": {"iters": [14] * 16, "s_per_rhs": 0.123456789, "top_kernels": {f"k{k}": {"avg_us": 1.0} for k in
                                                                                 range(40)}},
             "serving": {f"leg{k}": {"p50_ms": 22.9, "p99_ms": 96.91, "wall_s": 1.0, "not_ok": 0} for k in range(5)}}
    line = bench.result_line(RESULT, extra)
    assert "\n" not in line and len(line) <= bench.LINE_CHARS < 8000
    out = json.loads(line)
    assert {k: out[k] for k in RESULT} == RESULT
    assert out["extra"]["gspmv_chan256"]["f64/m3"] == [123.46, 4322.0]
    assert out["extra"]["amg"] == {"s_per_rhs": 0.12346} and "left_out" not in out["extra"]


def test_legs_that_do_not_fit_are_named():
    extra = {"iters_max": 5, "large": {str(k): 0.1 for k in range(5000)}, "small": {"a": 1}}
    out = json.loads(bench.result_line(RESULT, extra))
    assert out["extra"] == {"iters_max": 5, "small": {"a": 1}, "left_out": ["large"]}
    assert out["value"] == RESULT["value"]
