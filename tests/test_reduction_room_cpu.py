"""The partial sums of a reduction must stay clear of the column tickets, which
live in the second half of the same buffer: a reduction of more than 64 values
per workgroup (five dots of sixteen columns) must not compile, and what the
library has (four dots of sixteen columns, eight of eight) must."""
import subprocess

import pytest

from paper_1711_10622_amd import build

SOURCE = """
#include "internal.h"
struct Probe {
    static constexpr int NDOT = %d;
    __device__ void finish(const double *) const {}
};
__global__ void k(mrhs::RedBufs<double> rb)
{
    mrhs::Acc<double, mrhs::Shape<double, %d>::VW, Probe::NDOT> acc;
    acc.zero();
    mrhs::grid_reduce<double, %d, Probe::NDOT>(acc, rb, Probe{});
}
"""


@pytest.mark.parametrize("ndot,m,fits", [(4, 16, True), (8, 8, True), (8, 1, True), (5, 16, False), (8, 9, False)])
def test_sums_stay_clear_of_the_tickets(tmp_path, ndot, m, fits):
    src = tmp_path / "probe.hip"
    src.write_text(SOURCE % (ndot, m, m))
    cmd = [build.hipcc(), *build.flags(), "--cuda-device-only", "-fsyntax-only", str(src)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert (r.returncode == 0) == fits, r.stderr[-2000:]
    if not fits:
        assert "column tickets" in r.stderr
