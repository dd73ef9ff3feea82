"""Which sweep the benchmark says it timed, checked without a GPU."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


class Handle:
    """The launches of a handle that marches `march` steps a launch, runs the
    blocked sweep of `halo` steps, or takes one launch per step (halo 1)."""

    def __init__(self, halo, march=0):
        self.halo, self.march, self.timed = halo, march, None

    def profile_sweeps(self, enable):
        out = self.timed
        self.timed = (0, 0, 0.0)
        return out

    def run(self, n, tol, k):
        assert tol == 0.0 and k == n
        launches = bench.march_launches(n, self.march) if self.march else -(-n // self.halo)
        self.timed = (n, launches, 1.0)


def test_march_launches():
    assert [bench.march_launches(100, s) for s in (1, 2, 4, 6, 7)] == [100, 50, 25, 17, 15]
    assert bench.march_launches(99, 4) == 24 + 2


@pytest.mark.parametrize("halo", [1, 2, 4, 8, 9])
def test_blocked_sweeps_are_told_apart_from_marching_ones(halo):
    assert bench.marching_steps(Handle(halo), halo) == 0
    for march in (4, 6, 7):
        assert bench.marching_steps(Handle(halo, march), halo) == march


def test_a_marching_launch_is_not_called_blocked():
    assert bench.kernel_label("f32", 7, 4, 16, 4, 6.7).startswith("march_kernel (f32 storage, 7 ")
    assert bench.kernel_label("f32", 0, 4, 16, 4, 4.0).startswith("tb_kernel (f32 storage, shape 4")
    assert bench.kernel_label("f32", 0, 4, 16, 4, 1.0).startswith("step_kernel")


def test_issue_rate_against_what_the_simds_reach():
    roof = {}
    bench.hbm_and_limiter(roof, None, 1.0e6, 0.0135, "f64")
    peak = 256 * 4 * 2.4e9 / 4.6
    assert roof["limiter"]["frac_of_measured_rate"] == pytest.approx(1.0e6 / 13.5e-6 / peak, rel=1e-3)
