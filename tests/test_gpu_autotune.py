"""What the autotuner picks on a handle that can run an iteration as one launch:
a variant those launches take (0, 8 or 9; learned: of the M^-1 product), unless
whole iterations with another product are faster -- a tuned handle's steps
are no slower than an untuned one's."""
import os
import time

import numpy as np
import pytest

from paper_1808_06381_amd import inputs, precond
from paper_1808_06381_amd import sim as S

pytestmark = pytest.mark.gpu
WEIGHTS = os.path.join(os.path.dirname(precond.__file__), "weights", "precond_n1e5.bin")


def steps_ms(sim, steps=20, rounds=5):
    best = np.inf
    for _ in range(rounds):
        t = time.perf_counter()
        for _ in range(steps):
            sim.step(1)
        best = min(best, time.perf_counter() - t)
    return best / steps * 1e3


@pytest.mark.parametrize("pc", ["jacobi", "none", "learned"])
def test_a_tuned_small_handle_keeps_its_fused_iterations(pc):
    cfg = inputs.cube_params(1000, 0.05, seed=1)
    pos = inputs.uniform_positions(1000, cfg["box"], 1)
    with S.Sim(cfg, pos, tol=1e-10, precond=pc) as sim, \
            S.Sim(cfg, pos, tol=1e-10, precond=pc) as plain:
        for s in (sim, plain):
            if pc == "learned":
                s.load_precond(WEIGHTS)
            s.graph_mode(True)
            s.step(3)
        t = sim.autotune(reps=10)
        for s in (sim, plain):
            s.step(5)   # records the graph
        a, b = steps_ms(sim), steps_ms(plain)
        assert t["apply_variant" if pc == "learned" else "spmv_variant"] in (0, 8, 9)
        # the same launches but for the order of columns ahead: noise only
        # (separate launches take more than 1.8 times as long)
        assert a <= 1.25 * b, (a, b, t)


@pytest.mark.parametrize("pc", ["jacobi", "none", "ic0", "learned"])
@pytest.mark.parametrize("n", [2000, 140_000])
def test_tuning_leaves_the_state_and_a_working_handle(n, pc):
    cfg = inputs.cube_params(n, 0.2, seed=2)
    pos = inputs.uniform_positions(n, cfg["box"], 2)
    with S.Sim(cfg, pos, tol=1e-9, precond=pc) as sim:
        if pc == "learned":
            sim.load_precond(WEIGHTS)
        sim.step(1)
        before = sim.state()
        t = sim.autotune(reps=3)
        after = sim.state()
        assert np.array_equal(before[0], after[0]) and np.array_equal(before[1], after[1])
        assert all(u > 0 for u in t["spmv_us"]) and all(u > 0 for u in t["vec_us"])
        st = sim.step(2)
        assert max(st["relres"]) <= 1e-9 and st["steps_done"] == 2 and st["fallback"] == 0


@pytest.mark.parametrize("n", [300, 1000, 4000, 20_000, 60_000, 131_072])
def test_the_vector_form_stays_where_no_launch_has_one(n):
    cfg = inputs.cube_params(n, 0.1, seed=4)
    with S.Sim(cfg, inputs.uniform_positions(n, cfg["box"], 4), tol=1e-8) as sim:
        t = sim.autotune(reps=3)
        assert t["spmv_variant"] not in (0, 8, 9) or t["vec_variant"] == 0


def test_tuning_a_system_that_needs_no_iterations():
    """Every product is the diagonal's and the right-hand side is zero."""
    cfg = dict(inputs.base_params(n=64, box=(40.0, 40.0, 40.0), shear_rate=0.0, seed=1), kT=0.0)
    g = (np.arange(4) + 0.5) * 10.0
    pos = np.stack(np.meshgrid(g, g, g), -1).reshape(-1, 3)
    with S.Sim(cfg, pos, tol=1e-9) as sim:
        t = sim.autotune(reps=2)
        assert t["spmv_variant"] in range(len(S.CSR_VARIANTS))
        sim.step(2)
        p, v, _ = sim.state()
    assert np.all(v == 0.0) and np.array_equal(p, pos)
