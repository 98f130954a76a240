"""Handles past the fused iterations' size advance the CG scalars in the vector
pass, from sums that a short launch leaves per group of sub-tiles.  They must
give the bits of the separate finisher, which the timing probe selects in
every other solve: one group and several, groups of 64 and of 128 sub-tiles,
uneven batches, replicas that finish early, rings that wrap."""
import numpy as np
import pytest

from paper_1808_06381_amd import inputs
from test_gpu_cg_fused import both

pytestmark = pytest.mark.gpu
SUB = 256


@pytest.mark.parametrize("n", [512 * SUB + 1, 512 * SUB + 64 * SUB + 1, 4096 * SUB, 4096 * SUB + 1])
@pytest.mark.parametrize("kw", [dict(), dict(precond="none"), dict(spmv_fp32=1),
                                dict(precond="learned")], ids=lambda k: str(k))
def test_single_box(n, kw):
    both([inputs.cube_params(n, 0.3, seed=2)], steps=2, tol=1e-8, **kw)


@pytest.mark.parametrize("pc", ["jacobi", "learned"])
def test_uneven_replicas(pc):
    cfgs = [dict(inputs.cube_params(n, 0.3 * (r + 1), seed=r), stream=r, gamma0=g)
            for r, (n, g) in enumerate([(700, 40.0), (140000, 1.0), (255, 0.05), (60000, 0.2)])]
    both(cfgs, steps=2, precond=pc)


def test_wrapping_ring_and_graph():
    from paper_1808_06381_amd import sim as S
    cfg = dict(inputs.cube_params(150000, 0.3, seed=4), gamma0=1e-3, alpha=4.0)
    its = both([cfg], steps=2, tol=1e-10)[2]
    assert max(max(i) for i in its) > 128
    pos = inputs.uniform_positions(cfg["n"], cfg["box"], 50)
    out = []
    for graph in (False, True):
        with S.Sim(cfg, pos, tol=1e-10) as sim:
            sim.graph_mode(graph)
            for _ in range(5):
                sim.step(1)
            out.append(sim.state()[:2])
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
