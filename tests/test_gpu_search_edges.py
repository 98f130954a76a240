"""The neighbour search and pair terms where their forms change: small handles
(sixteen lanes per particle, 64-row tiles of entries) against large ones,
boxes of three and four cells per axis (no cell away from the faces), a one-cell
axis, waves with and without particles at the faces, rows longer than a lane's
and the list's kept candidates, scans of one and several blocks.  Pair sets
bit-exact and the system against the oracle (A bit-exact for the polynomial
weight, b to 1e-11 of its largest entry, as in test_gpu_parity)."""
import numpy as np
import pytest

import oracle
from paper_1808_06381_amd import inputs
from paper_1808_06381_amd import sim as S

pytestmark = pytest.mark.gpu


def check(cfg, pos, steps=0):
    with S.Sim(cfg, pos, tol=1e-10) as sim:
        if steps:
            sim.step(steps)
        p = sim.state()[0]
        got = sim.pairs()
        rows, cols, vals, diag, rhs = sim.system()
    delta = oracle.le_offset(cfg, steps)
    ref = np.asarray(oracle.pairs(cfg, p, delta, method="cells" if cfg["n"] > 4000 else "brute"))
    ref = ref[:, -2:]
    ref = ref[np.lexsort((ref[:, 1], ref[:, 0]))]
    assert np.array_equal(got[:, 1:], ref)
    s = oracle.build_system(cfg, p, steps)
    assert len(vals) == 2 * len(ref)
    assert np.max(np.abs(rhs - s["rhs"])) <= 1e-11 * np.max(np.abs(s["rhs"]))
    # row sums of the off-diagonal part and the diagonal (sums in another order)
    assert np.allclose(diag, s["diag"], rtol=1e-13, atol=0)
    off = np.zeros(cfg["n"])
    np.add.at(off, rows, vals)
    assert np.allclose(cfg["gamma0"] - off, diag, rtol=1e-12, atol=0)


@pytest.mark.parametrize("cells", [(3, 3, 3), (4, 3, 5), (1, 4, 4), (4, 1, 4), (4, 4, 1), (9, 8, 7)])
@pytest.mark.parametrize("density,steps", [(1.0, 0), (6.0, 2), (40.0, 1)])
def test_box_shapes(cells, density, steps):
    box = tuple(2.05 if c == 1 else c * 1.01 for c in cells)
    n = max(3, int(density * np.prod(box)))
    cfg = inputs.base_params(n=n, box=box, shear_rate=0.7, seed=n)
    check(cfg, inputs.uniform_positions(n, box, n), steps)


def test_long_rows_of_one_cell():
    # every particle of a clump is every other's neighbour: 200-entry rows
    cfg = inputs.base_params(n=700, box=(8.0, 8.0, 8.0), shear_rate=0.2, seed=4)
    pos = inputs.uniform_positions(700, cfg["box"], 4)
    pos[:200] = 4.0 + 0.3 * (pos[:200] / 8.0 - 0.5)
    check(cfg, pos)


@pytest.mark.parametrize("n", [7000, 8191, 131072, 131073, 140000])
def test_handle_sizes(n):
    cfg = inputs.cube_params(n, 0.5, seed=n)
    check(cfg, inputs.uniform_positions(n, cfg["box"], n), 0 if n > 10000 else 2)
