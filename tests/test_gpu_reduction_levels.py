"""The CG's partial sums on both sides of the line from which several blocks
share a replica's reduction (more than 512 sub-tiles of 256 rows), scalar and
block system, alone and next to a small replica.

Oracle: the residual of the returned solution, formed on the host from the
exported system, is at most tol plus the rounding of that product; and a
replica's bits do not depend on the batch (nor on which block came last).
"""
import numpy as np
import pytest

from paper_1808_06381_amd import inputs
from paper_1808_06381_amd import sim as S

pytestmark = pytest.mark.gpu
LINE = 512 * 256


@pytest.mark.parametrize("n", [LINE, LINE + 1, LINE + 65 * 256, 4 * LINE + 257])
def test_scalar_system(n):
    cfg = dict(inputs.cube_params(n, 0.3, seed=2), stream=0)
    small = dict(inputs.cube_params(700, 0.3, seed=3), stream=1)
    pos = [inputs.uniform_positions(c["n"], c["box"], 4 + i) for i, c in enumerate((cfg, small))]
    b = [np.random.default_rng(i).normal(size=(c["n"], 3)) for i, c in enumerate((cfg, small))]
    tol = 1e-9
    with S.Sim(cfg, pos[0], tol=tol) as sim:
        v, st = sim.solve(b[0])
        again, _ = sim.solve(b[0])
        rows, cols, vals, diag, _ = sim.system()
    assert np.array_equal(v, again)
    Av, Aa = np.empty_like(v), np.empty_like(v)
    for k in range(3):
        Av[:, k] = diag * v[:, k] + np.bincount(rows, vals * v[cols, k], n)
        Aa[:, k] = np.abs(diag * v[:, k]) + np.bincount(rows, np.abs(vals * v[cols, k]), n)
    bn = np.linalg.norm(b[0], axis=0)
    slack = 64 * np.finfo(float).eps * np.linalg.norm(Aa, axis=0) / bn
    assert np.all(np.linalg.norm(b[0] - Av, axis=0) / bn <= tol + slack)
    with S.Sim([cfg, small], np.concatenate(pos), tol=tol) as sim:
        both, _ = sim.solve(np.concatenate(b))
    assert np.array_equal(both[:n], v)


@pytest.mark.parametrize("n", [LINE, LINE + 257])
def test_block_system(n):
    cfg = dict(inputs.cube_params(n, 0.3, seed=5), friction_par=1.5, friction_perp=0.5, stream=0)
    small = dict(cfg, n=900, box=inputs.cube_params(900, 0.3, seed=5)["box"], stream=1)
    pos = [inputs.uniform_positions(c["n"], c["box"], 8 + i) for i, c in enumerate((cfg, small))]
    b = [np.random.default_rng(9 + i).normal(size=(c["n"], 3)) for i, c in enumerate((cfg, small))]
    tol = 1e-9
    with S.Sim(cfg, pos[0], tol=tol) as sim:
        v, st = sim.solve(b[0])
    assert st["relres"][0] <= tol and np.all(np.isfinite(v))
    with S.Sim([cfg, small], np.concatenate(pos), tol=tol) as sim:
        both, _ = sim.solve(np.concatenate(b))
    assert np.array_equal(both[:n], v)
