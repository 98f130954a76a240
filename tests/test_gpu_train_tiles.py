"""The training backward pass at the edges of its tiles: rows of one and of
several 64-row tiles per block, tiles whose entries need several stages in LDS
(dense boxes), and the two sums over blocks.  Gradients of every parameter
tensor against the FP64 oracle on the same weights, with the tolerances of
test_gpu_learned (FP32 sums against FP64: 1e-3 of the tensor's norm plus 1e-7
of the whole gradient's)."""
import numpy as np
import pytest

import oracle
from paper_1808_06381_amd import inputs
from paper_1808_06381_amd import sim as S
from test_gpu_learned import assert_grad_per_tensor, oracle_probe, random_theta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,density", [(63, 1.0), (65, 1.0), (1100, 10.0), (2500, 30.0)])
def test_gradient_tiles(n, density):
    cfg = inputs.cube_params(n, 0.2, seed=n, density=density)
    if min(cfg["box"]) <= 2.0:
        cfg = dict(cfg, rc=0.45 * min(cfg["box"]))
    pos = inputs.uniform_positions(n, cfg["box"], n)
    th = random_theta(7)
    with S.Sim(cfg, pos, tol=1e-10) as sim:
        sim.set_weights(th)
        sim.precond_config(round_act=False)
        st = sim.step(0)
        sim.solve(np.random.default_rng(1).normal(size=(n, 3)))
        loss = sim.train_probe(0.0, seed=7, index=2)
        g = sim.precond_grad().astype(np.float64)
        again = sim.train_probe(0.0, seed=7, index=2)
        assert again == loss and np.array_equal(g, sim.precond_grad())
    s = oracle.build_system(cfg, pos, 0)
    er = oracle.edge_r(cfg, pos, s, 0)
    z = oracle_probe(cfg, 7, 2)
    lo, go = oracle.mpnn_loss_grad(s, er, cfg["alpha"], th, oracle.spmv3(s, z), z, norm="2")
    assert loss == pytest.approx(lo, rel=1e-4)
    assert np.linalg.norm(g - go) <= 1e-3 * np.linalg.norm(go)
    assert_grad_per_tensor(g, go)
    del st


def test_several_tiles_per_block():
    """4200 tiles and more, so that a block of the layers' backward walks two:
    a batch of copies of one box must give the gradient of that box (the loss
    is a ratio of sums over replicas that all agree, their probes keyed by the
    same stream), to FP32 rounding of the sums: 1e-4 of each tensor's norm
    allows 2^-24 times the square root of 3e5 rows with a factor of three."""
    n, copies = 5000, 54          # 54 x 80 tiles of 64 rows
    cfg = dict(inputs.cube_params(n, 0.2, seed=3), stream=0)
    pos = inputs.uniform_positions(n, cfg["box"], 3)
    th = random_theta(4)
    out = []
    for c in (1, copies):
        with S.Sim([dict(cfg)] * c, np.concatenate([pos] * c), tol=1e-8) as sim:
            sim.set_weights(th)
            sim.step(1)
            loss = sim.train_probe(0.0, seed=5, index=1)
            out.append((loss, sim.precond_grad().astype(np.float64)))
    assert out[1][0] == pytest.approx(out[0][0], rel=1e-10)
    from paper_1808_06381_amd import precond
    for name, (off, shape) in precond.LAYOUT.items():
        a, b = (o[1][off:off + int(np.prod(shape))] for o in out)
        assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(a) + 1e-7 * np.linalg.norm(out[0][1]), name
