"""Structure factor at the edges of the contraction's tiles: 64 mx and 64 my
values per block, 16 x 16 per wave, 32 particles per table group, chunks of
4096 rows; the mirrored half my < 0 and my = 0 come from the same sums.  Every
output against the oracle, tolerance as derived in test_gpu_sq (phases to
2 pi |m| 4 eps, tables to 16 eps, twice that bound)."""
import numpy as np
import pytest

from paper_1808_06381_amd import inputs
from paper_1808_06381_amd import sim as S
from test_gpu_sq import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [9, 31, 32, 33, 4097])
@pytest.mark.parametrize("nx,my_max,mz", [(1, 0, 0), (16, 0, 3), (17, 1, 0), (64, 16, 2),
                                          (65, 17, -5), (5, 64, 1), (48, 65, 0), (80, 80, 0),
                                          (33, 128, 7)])
def test_tile_edges(n, nx, my_max, mz):
    cfg = inputs.cube_params(n, 0.6, seed=n)
    pos0 = inputs.uniform_positions(n, cfg["box"], n)
    with S.Sim(cfg, pos0) as sim:
        sim.step(2)
        pos, _, _ = sim.state()
        got = sim.structure_factor(nx, my_max, mz=mz)
    assert got.shape == (1, nx, 2 * my_max + 1)
    check(cfg, pos, 2, got[0], nx, my_max, mz)
    if mz == 0 and nx > 0:   # S(-q) = S(q) on the mx = 0 line
        assert np.allclose(got[0, 0], got[0, 0, ::-1], rtol=1e-12, atol=1e-12)
