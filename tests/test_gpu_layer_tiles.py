"""The network's layers on the matrix cores at the edges of their tiles: rows
without neighbours, groups of four entries exactly and partly filled, tiles of
more than 128 groups (several passes), handles of one and several row blocks.
M^-1 against the oracle on the same bfloat16 weights; activations are rounded
to bfloat16, so 3e-2 relative as in test_gpu_learned."""
import numpy as np
import pytest

from paper_1808_06381_amd import inputs
from paper_1808_06381_amd import sim as S
from test_gpu_learned import oracle_minv, random_theta, sorted_triples

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,density", [(40, 0.02), (64, 1.0), (65, 1.0), (1000, 0.3), (1100, 12.0),
                                       (3000, 40.0)])
def test_minv(n, density):
    cfg = inputs.cube_params(n, 0.2, seed=n, density=density)
    pos = inputs.uniform_positions(n, cfg["box"], n)
    th = random_theta(2)
    with S.Sim(cfg, pos, precond="learned") as sim:
        sim.set_weights(th)
        gr, gc, gv, gd = sim.precond_matrix()
    s, er, md, orow, ocol, ov = oracle_minv(cfg, pos, th)
    gr, gc, gv = sorted_triples(gr, gc, gv)
    orow, ocol, ov = sorted_triples(orow, ocol, ov)
    assert np.array_equal(gr, orow) and np.array_equal(gc, ocol)
    np.testing.assert_allclose(gd, md, rtol=3e-2)
    if len(ov):
        np.testing.assert_allclose(gv, ov, rtol=3e-2, atol=3e-2 * np.abs(ov).max())
