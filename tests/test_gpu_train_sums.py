"""The parameter gradient's sum over the rows of a large system: every 64-row
tile leaves its own FP32 sums and these are added in FP64, so a batch of
copies of one box must give that box's gradient to the last rounding.

The loss is a ratio of sums over replicas that all agree, and a replica's rows
and its probe do not depend on the rest of the batch, so every copy leaves
the tile sums of the single box.  Both gradients are FP64 totals of those,
the batch's the number of copies times the other's, scaled and rounded to
FP32 once: per element they differ by two roundings (2^-24 each; 2^-22
allows for the scaling), also where the tiles nearly cancel, plus 2^-53 per
addition of a tile sum: 1e-12 of the tensor's norm allows tile sums of that
norm times 50.  FP32 sums over several tiles miss this by far where tiles
cancel."""
import numpy as np
import pytest

from paper_1808_06381_amd import inputs, precond
from paper_1808_06381_amd import sim as S
from test_gpu_learned import random_theta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("round_act", [True, False])
def test_copies_give_the_gradient_of_one(round_act):
    n, copies = 5000, 54          # 54 x 80 tiles of 64 rows
    cfg = dict(inputs.cube_params(n, 0.2, seed=3), stream=0)
    pos = inputs.uniform_positions(n, cfg["box"], 3)
    th = random_theta(4)
    g = []
    for c in (1, copies):
        with S.Sim([dict(cfg)] * c, np.concatenate([pos] * c), tol=1e-8) as sim:
            sim.set_weights(th)
            sim.precond_config(round_act=round_act)
            sim.step(1)
            sim.train_probe(0.0, seed=5, index=1)
            g.append(sim.precond_grad().astype(np.float64))
    for name, (off, shape) in precond.LAYOUT.items():
        a, b = (x[off:off + int(np.prod(shape))] for x in g)
        assert np.all(np.abs(a - b) <= 2.0 ** -22 * np.abs(a) + 1e-12 * np.linalg.norm(a)), \
            (name, float(np.max(np.abs(a - b) / np.maximum(np.abs(a), 1e-30))))
