"""The scalar CG's ring of preconditioned residuals where it can go wrong:
solves longer than the ring's 64 slots (the ring wraps, several passes over
x), components and replicas of one handle that finish at very different
iterations (terms pending while others wrap), every preconditioner, restarts
after a failed check, and steps that continue past a recorded graph.

Oracle: a dense solve; with the true residual at or below tol the relative
error of every component is at most cond(A) * tol.
"""
import os

import numpy as np
import pytest

import oracle
from paper_1808_06381_amd import inputs, precond
from paper_1808_06381_amd import sim as S

pytestmark = pytest.mark.gpu
WEIGHTS = os.path.join(os.path.dirname(precond.__file__), "weights", "precond_n1e5.bin")


def stiff(n, gamma0, seed):
    """A box whose friction system needs hundreds of Jacobi iterations."""
    c = inputs.cube_params(n, 0.3, seed=seed, density=2.0)
    return dict(c, gamma0=gamma0, alpha=4.0)


def dense_of(cfg, pos):
    return oracle.dense(oracle.build_system(cfg, pos, 0))


@pytest.mark.parametrize("pc", ["jacobi", "none", "ic0", "learned"])
@pytest.mark.parametrize("gamma0", [1e-1, 1e-3, 1e-5])
def test_solves_longer_than_the_ring(pc, gamma0):
    cfg = stiff(1500, gamma0, 5)
    pos = inputs.uniform_positions(cfg["n"], cfg["box"], 5)
    A = dense_of(cfg, pos)
    rng = np.random.default_rng(2)
    b = rng.normal(size=(cfg["n"], 3))
    b[:, 1] = A @ np.ones(cfg["n"])       # the smoothest mode: the last to converge
    x = np.linalg.solve(A, b)
    tol = 1e-10
    with S.Sim(cfg, pos, tol=tol, precond=pc) as sim:
        if pc == "learned":
            sim.load_precond(WEIGHTS)
        v, st = sim.solve(b)
        v2, st2 = sim.solve(b)
    if gamma0 <= 1e-3 and pc in ("jacobi", "none"):
        assert max(st["iters"]) > 128      # two wraps at least
    err = np.linalg.norm(v - x, axis=0) / np.linalg.norm(x, axis=0)
    assert np.all(err <= np.linalg.cond(A) * tol), (err, st)
    assert max(st["relres"]) <= tol
    # the second solve polls at other iterations (its first chunk is longer), so
    # a learned solve may stall, and be redone with Jacobi, in one of the two only
    if st2["fallback"] == st["fallback"]:
        assert np.array_equal(v, v2)


def test_replicas_and_components_that_finish_far_apart():
    """One replica needs a few iterations, one hundreds; in both a component
    with b = 0.  A replica's bits do not depend on the rest of the batch."""
    cfgs = [dict(stiff(900, 50.0, 3), stream=0), dict(stiff(1100, 1e-4, 4), stream=1)]
    pos = [inputs.uniform_positions(c["n"], c["box"], 30 + r) for r, c in enumerate(cfgs)]
    rng = np.random.default_rng(8)
    b = [rng.normal(size=(c["n"], 3)) for c in cfgs]
    b[0][:, 2] = 0.0
    b[1][:, 0] = 0.0
    tol = 1e-10
    with S.Sim(cfgs, np.concatenate(pos), tol=tol) as sim:
        v, st = sim.solve(np.concatenate(b))
    parts = np.split(v, [cfgs[0]["n"]])
    for c, p, bb, vv in zip(cfgs, pos, b, parts):
        A = dense_of(c, p)
        x = np.linalg.solve(A, bb)
        zero = np.all(bb == 0.0, axis=0)
        assert np.all(vv[:, zero] == 0.0)
        err = np.linalg.norm((vv - x)[:, ~zero], axis=0) / np.linalg.norm(x[:, ~zero], axis=0)
        assert np.all(err <= np.linalg.cond(A) * tol), err
        with S.Sim(c, p, tol=tol) as one:
            alone, st1 = one.solve(bb)
        assert np.array_equal(alone, vv)
    assert max(st["iters"]) > 128


def test_restart_after_a_failed_check():
    """A tolerance near the rounding level of a stiff system: the recursive
    residual passes before the true one, components restart, and the final
    true residual (formed here) meets the tolerance or the solve says so."""
    cfg = stiff(1200, 1e-4, 9)
    pos = inputs.uniform_positions(cfg["n"], cfg["box"], 9)
    A = dense_of(cfg, pos)
    b = np.random.default_rng(4).normal(size=(cfg["n"], 3))
    for tol in (1e-12, 3e-14):
        with S.Sim(cfg, pos, tol=tol, maxit=4000) as sim:
            try:
                v, st = sim.solve(b)
            except S.SimError as e:
                assert tol < 1e-13 and e.code in (-4, -5)
                continue
        res = np.linalg.norm(b - A @ v, axis=0) / np.linalg.norm(b, axis=0)
        # numpy's own product rounds at cond-independent ~n eps |A||v| / |b|
        slack = 64 * np.finfo(float).eps * np.linalg.norm(np.abs(A) @ np.abs(v), axis=0) \
            / np.linalg.norm(b, axis=0)
        assert np.all(res <= tol + slack), (tol, res, st)


def test_graph_steps_past_the_ring_bitwise_equal_eager():
    cfg = stiff(1300, 1e-3, 12)
    pos = inputs.uniform_positions(cfg["n"], cfg["box"], 12)
    out = []
    for graph in (False, True):
        with S.Sim(cfg, pos, tol=1e-10) as sim:
            sim.graph_mode(graph)
            its = [max(sim.step(1)["iters"]) for _ in range(6)]
            out.append(sim.state()[:2] + (its,))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert out[0][2] == out[1][2] and max(its) > 128


@pytest.mark.parametrize("pc", ["jacobi", "learned"])
@pytest.mark.parametrize("gamma0", [1e-1, 1e-3])
def test_block_solves_longer_than_the_ring(pc, gamma0):
    """The block system's ring, alone and in a batch with a replica that
    finishes early; the same bound with the stacked residual."""
    cfgs = [dict(stiff(700, gamma0, 6), friction_par=2.0, friction_perp=0.5, stream=0),
            dict(inputs.cube_params(500, 0.2, seed=7), gamma0=50.0, friction_par=0.5,
                 friction_perp=1.5, stream=1)]
    pos = [inputs.uniform_positions(c["n"], c["box"], 70 + r) for r, c in enumerate(cfgs)]
    b = [np.random.default_rng(r).normal(size=(c["n"], 3)) for r, c in enumerate(cfgs)]
    tol = 1e-10
    with S.Sim(cfgs, np.concatenate(pos), tol=tol, precond=pc) as sim:
        if pc == "learned":
            sim.set_weights(precond.block_params(precond.load(WEIGHTS)))
        v, st = sim.solve(np.concatenate(b))
    for c, p, bb, vv in zip(cfgs, pos, b, np.split(v, [cfgs[0]["n"]])):
        A = oracle.block_dense(oracle.build_block_system(c, p, c["friction_par"], c["friction_perp"]))
        x = np.linalg.solve(A, bb.reshape(-1))
        err = np.linalg.norm(vv.reshape(-1) - x) / np.linalg.norm(x)
        assert err <= np.linalg.cond(A) * tol, (err, st)
    if gamma0 < 1e-2 and not st["fallback"] and pc == "jacobi":
        assert max(st["iters"]) > 128
