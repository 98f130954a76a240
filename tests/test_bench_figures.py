"""Figures that bench.py derives (CPU): the structure factor's operations are
those the contraction performs."""
import numpy as np
import pytest

import bench


class FakeSim:
    """A handle whose structure factor takes 2 ms."""

    def structure_factor(self, nx, my_max, timed=False):
        s = np.ones((1, nx, 2 * my_max + 1))
        return (s, 2.0) if timed else s


def test_structure_factor_operations():
    """Four real sums of products (P1 .. P4: 8 flops) give rho at (mx, my) and
    at (mx, -my), and my = 0 is a sum of two: per mx 8 my_max + 2 flops for
    2 my_max + 1 wavevectors, so 4 per wavevector but for a part in my_max."""
    n, nx, my_max = 1000, 64, 64
    r = bench.measure_sq(FakeSim(), n, np, nx, my_max)
    assert r["kernel_ms_events"] == 2.0
    assert r["flops_per_call"] == 4.0 * n * nx * (2 * my_max + 1)
    assert r["flops_per_call"] == pytest.approx(n * nx * (8 * my_max + 2), rel=0.5 / my_max)
