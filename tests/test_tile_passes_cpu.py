"""Where a full tile is one pass of the workgroup the compiler must know it: the
passes per tile are then a constant expression whatever the launch says (a
run-time loop made products of one binary64 column up to 70 % slower on
multigrid levels), and elsewhere the launch's own count."""
import subprocess

import pytest

from paper_1711_10622_amd import build

SOURCE = """
#include "core.h"
using S = mrhs::Shape<%s, %d>;
constexpr mrhs::TilePlan launch{2, 1};
static_assert(S::PASSES %s 1, "");
static_assert(mrhs::plan_passes<S>(launch) == %d, "passes of the tile");
"""


@pytest.mark.parametrize("t,m", [("double", 1), ("double", 2), ("float", 1), ("float", 2), ("float", 4)])
def test_one_pass_is_a_constant(tmp_path, t, m):
    assert compiles(tmp_path, SOURCE % (t, m, "==", 1))


@pytest.mark.parametrize("t,m", [("double", 4), ("double", 9), ("double", 16), ("float", 8), ("float", 16)])
def test_other_tiles_follow_the_launch(tmp_path, t, m):
    assert compiles(tmp_path, SOURCE % (t, m, ">", 2))


@pytest.mark.parametrize("ndot,passes", [(0, "S::PASSES"), (1, "2")])
def test_products_without_a_reduction_take_full_tiles(tmp_path, ndot, passes):
    assert compiles(tmp_path, f"""
#include "core.h"
using S = mrhs::Shape<double, 9>;
struct Op {{ static constexpr int NDOT = {ndot}; }};
constexpr mrhs::TilePlan launch{{2, 1}};
static_assert(mrhs::plan_passes<S, Op>(launch) == {passes}, "passes of the tile");
""")


def compiles(tmp_path, text):
    src = tmp_path / "probe.hip"
    src.write_text(text)
    r = subprocess.run([build.hipcc(), *build.flags(), "--cuda-host-only", "-fsyntax-only", str(src)],
                       capture_output=True, text=True)
    assert "fatal" not in r.stderr
    return r.returncode == 0 or pytest.fail(r.stderr[-1500:])


@pytest.mark.parametrize("n,rows,full,passes", [(1, 32, 8, 1), (8192, 32, 8, 1), (8193, 32, 8, 2), (32768, 32, 8, 4),
                                                (53760, 64, 4, 4), (53760, 32, 8, 7), (65537, 32, 8, 8),
                                                (12582912, 32, 8, 8), (2147483647, 256, 1, 1)])
def test_no_unit_gets_two_tiles(tmp_path, n, rows, full, passes):
    """A reducing kernel's tiles on 256 compute units: no more tiles than units
    as long as a full tile allows it."""
    assert compiles(tmp_path, f"""
#include "internal.h"
static_assert(mrhs::balanced_passes({n}, 256, {rows}, {full}) == {passes}, "passes");
""")
    assert passes == full or -(-n // (passes * rows)) <= 256
