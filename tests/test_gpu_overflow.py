"""Neighbour lists that do not fit: offsets past the 32-bit range never decrease
(so that a clamped reader stays in bounds) and are reported, and a box whose
clusters need several times the list's first capacity gives the oracle's pairs,
system and steps, eagerly and with step graphs."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from paper_1808_06381_amd import inputs
from paper_1808_06381_amd import sim as S

pytestmark = pytest.mark.gpu


def scan(v):
    """The library's exclusive scan (internal, reached by its C++ name)."""
    fn = getattr(S.lib(), "_Z11launch_scanPKiPilS1_P12ihipStream_tS1_")
    fn.argtypes = [C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p]
    n = len(v)
    a = torch.from_numpy(np.asarray(v, np.int32)).cuda()
    out = torch.full((n + 8,), -7, dtype=torch.int32, device="cuda")
    bsum = torch.zeros(n // 8192 + 2, dtype=torch.int32, device="cuda")
    many = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert fn(a.data_ptr(), out.data_ptr(), n, bsum.data_ptr(), None, many.data_ptr()) == 0
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(got[n:] == -7)
    return got[:n], int(many.item())


@pytest.mark.parametrize("n", [1, 7, 8, 511, 8191, 8192, 8193, 16384, 40001, 300_000])
@pytest.mark.parametrize("most", [3, 20_000, 400_000, 2**31 - 1])
def test_scan_saturates(n, most):
    v = np.random.default_rng(n).integers(0, most, size=n, endpoint=True)
    want = np.concatenate([[0], np.cumsum(v, dtype=np.int64)])
    got, many = scan(v)
    assert np.array_equal(got, np.minimum(want[:-1], 2**31 - 1))
    assert many == int(want[-1] > 2**31 - 1)


def clustered(n, box, radius, seed):
    rng = np.random.default_rng(seed)
    return np.asarray(box) / 2 + rng.uniform(-radius, radius, size=(n, 3))


@pytest.mark.parametrize("n", [700, 3000])
@pytest.mark.parametrize("graph", [False, True])
def test_a_cluster_grows_the_list(n, graph):
    # about n / 6 neighbours per particle, room for 17: several growths' worth
    cfg = inputs.base_params(n=n, box=(30.0, 30.0, 30.0), shear_rate=0.2, seed=3)
    pos = clustered(n, cfg["box"], 0.8, 3)
    steps = 2
    with S.Sim(cfg, pos, tol=1e-10) as sim:
        sim.graph_mode(graph)
        st = sim.step(steps)
        p, v, _ = sim.state()
        assert st["max_row"] > 100
    po, vo, _ = oracle.run(cfg, pos, steps, tol=1e-10)
    assert np.linalg.norm(v - vo) <= 1e-6 * np.linalg.norm(vo)
    assert np.max(np.abs(p - po)) <= 1e-6


def test_pairs_of_a_cluster_are_the_oracles():
    n = 1500
    cfg = inputs.base_params(n=n, box=(30.0, 30.0, 30.0), shear_rate=0.0, seed=3)
    pos = clustered(n, cfg["box"], 0.7, 5)
    with S.Sim(cfg, pos) as sim:
        got = sim.pairs()[:, 1:]
    d = pos[:, None, :] - pos[None, :, :]
    r2 = (d[..., 0] ** 2 + d[..., 1] ** 2) + d[..., 2] ** 2
    want = {(i, j) for i, j in zip(*np.nonzero(np.triu(r2 < cfg["rc"] ** 2, 1)))}
    assert {(min(i, j), max(i, j)) for i, j in got} == want
