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
    cfg = inputs.cube_params(N, 0.2, seed=1)
    with S.Sim(cfg, inputs.uniform_positions(N, cfg["box"], 1), tol=1e-9, precond=pc,
               spmv_fp32=fp32) as sim:
        if pc == "learned":
            sim.load_precond(WEIGHTS)
        sim.step(1)
        sim.profile_enable(1)
        for k in range(6):
            st = sim.solve(np.random.default_rng(k).normal(size=(N, 3)))[1]
        rec = sim.profile_read()
    per = {k: v["bytes"] / v["launches"] for k, v in rec.items() if v["launches"]}
    return per, st["nnz"]


# the last two residuals and w read, the new residual written: 96 B per row;
# where the kernel forms u itself 24 more, and with Jacobi 8 for 1/diag
@pytest.mark.parametrize("pc,row,sums", [("jacobi", 128, 6), ("none", 120, 6), ("ic0", 96, 3),
                                         ("learned", 96, 3)])
def test_vector_kernel(pc, row, sums):
    per, _ = probed(pc)
    assert per["k_cg_vec"] == pytest.approx(row * ROWS + sums * 8 * SLOTS, rel=1e-12)


@pytest.mark.parametrize("pc,fp32,row,entry", [
    ("jacobi", 0, 128 + 60, 12), ("jacobi", 1, 128 + 60, 8), ("none", 0, 120 + 60, 12),
    ("ic0", 0, 96 + 60 + 128, 12 + 12), ("learned", 0, 96 + 60 + 60, 12 + 8)])
def test_iteration(pc, fp32, row, entry):
    per, nnz = probed(pc, fp32)
    assert per["cg_iteration"] == pytest.approx(row * N + entry * nnz, rel=1e-12)
    # the passes by themselves (over the padded rows, with their partial sums)
    parts = sum(per.get(k, 0.0) for k in ("k_cg_vec", "k_cg_spmv", "k_cg_apply"))
    if pc != "ic0":
        assert per["cg_iteration"] < parts < 1.04 * per["cg_iteration"]
