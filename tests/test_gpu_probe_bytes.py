"""The timing probe's algorithmic bytes: what each launch has to read and write
in the form the handle runs."""
import os

import numpy as np
import pytest

from paper_1808_06381_amd import inputs, precond
from paper_1808_06381_amd import sim as S

pytestmark = pytest.mark.gpu
WEIGHTS = os.path.join(os.path.dirname(precond.__file__), "weights", "precond_n1e5.bin")
N = 5000
ROWS = 5120                      # padded to whole 1024-row tiles
SLOTS = ROWS // 256              # partial sums of a sub-tile, 8 B each


def probed(pc, fp32=0):
    """(bytes per launch, bytes of each run of iterations and its length, nnz)"""
    cfg = inputs.cube_params(N, 0.2, seed=1)
    per, runs = {}, []
    with S.Sim(cfg, inputs.uniform_positions(N, cfg["box"], 1), tol=1e-9, precond=pc,
               spmv_fp32=fp32) as sim:
        if pc == "learned":
            sim.load_precond(WEIGHTS)
        sim.step(1)
        sim.profile_enable(1)
        for k in range(6):
            st = sim.solve(np.random.default_rng(k).normal(size=(N, 3)))[1]
            for name, v in sim.profile_read().items():
                if not v["launches"]:
                    continue
                if name == "cg_iteration":
                    runs.append((v["launches"], v["bytes"]))
                else:
                    per[name] = v["bytes"] / v["launches"]
    return per, runs, st["nnz"]


def ring_passes(m, n):
    """Bytes of the passes over x in a run of m iterations with a ring of 64: 63
    terms, x read and written, the direction written (and read, after the
    first)."""
    passes = (m - 1) // 63
    return n * (passes * (24 * 63 + 72) + 24 * max(passes - 1, 0))


# the last two residuals and w read, the new residual written: 96 B per row;
# where the kernel forms u itself 24 more, and with Jacobi 8 for 1/diag
@pytest.mark.parametrize("pc,row,sums", [("jacobi", 128, 6), ("none", 120, 6), ("ic0", 96, 3),
                                         ("learned", 96, 3)])
def test_vector_kernel(pc, row, sums):
    per, _, _ = probed(pc)
    assert per["k_cg_vec"] == pytest.approx(row * ROWS + sums * 8 * SLOTS, rel=1e-12)


@pytest.mark.parametrize("pc,fp32,row,entry", [
    ("jacobi", 0, 128 + 60, 12), ("jacobi", 1, 128 + 60, 8), ("none", 0, 120 + 60, 12),
    ("ic0", 0, 96 + 60 + 128, 12 + 12), ("learned", 0, 96 + 60 + 60, 12 + 8)])
def test_iteration(pc, fp32, row, entry):
    per, runs, nnz = probed(pc, fp32)
    one = row * N + entry * nnz
    assert len(runs) == 3
    for m, total in runs:
        assert total == pytest.approx(m * one + ring_passes(m, N), rel=1e-12)
    # the passes by themselves (over the padded rows, with their partial sums)
    parts = sum(per.get(k, 0.0) for k in ("k_cg_vec", "k_cg_spmv", "k_cg_apply"))
    if pc != "ic0":
        assert one < parts < 1.04 * one


def test_iterations_that_fill_the_ring():
    """A run of more than 126 iterations holds two passes of a ring of 64."""
    n = 1200
    cfg = dict(inputs.cube_params(n, 0.3, seed=9, density=2.0), gamma0=1e-4, alpha=4.0)
    b = np.random.default_rng(4).normal(size=(n, 3))
    with S.Sim(cfg, inputs.uniform_positions(n, cfg["box"], 9), tol=1e-10) as sim:
        sim.solve(b)                    # the next solve's first chunk is as long
        sim.profile_enable(1)
        sim.solve(b)                    # launch by launch
        sim.profile_read()
        st = sim.solve(b)[1]            # as runs of iterations
        rec = sim.profile_read()["cg_iteration"]
    m = rec["launches"]
    assert m > 126
    want = m * (188 * n + 12 * st["nnz"]) + ring_passes(m, n)
    assert rec["bytes"] == pytest.approx(want, rel=1e-12)
