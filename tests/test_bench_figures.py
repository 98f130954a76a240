"""Figures that bench.py derives (CPU): the structure factor's operations are
those the contraction performs; the iteration's textbook count beside the
bytes that its passes move."""
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


def test_textbook_count_beside_the_moved_bytes():
    k, n = 5.5, 1000
    assert bench.textbook_bytes(k, n, False) == n * (12 * (k + 1) + 4 + 200)
    assert bench.textbook_bytes(k, n, True) == n * (2 * (12 * (k + 1) + 4) + 200)
    moved = n * (96 + 60 + 12 * k + 60 + 8 * k)
    it = dict(gbs=moved / 500.0 / 1e3, bytes_per_launch=moved, mean_us=500.0, launches=9)
    r = dict(rows=dict(mean_offdiag_per_row=k), particles=n,
             kernels=dict(cg_iteration=it, k_cg_apply=dict(it, mean_us=200.0)))
    out = bench.iteration_roofline(r, 5000.0, None)
    assert out["bytes_per_iteration"] == moved
    assert out["textbook_pcg_bytes"] == bench.textbook_bytes(k, n, True)
    assert out["frac"] == pytest.approx(moved / 500.0 / 1e3 / 8000.0, abs=1e-4)
    assert "60+12k" in out["basis"] and "200" not in out["basis"]
