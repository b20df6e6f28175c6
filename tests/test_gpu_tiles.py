"""The 2D tile kernel (several steps per launch on small grids, taken when no
tile is set) against the strips (any tile set): the same bits in the same
buffer, at grids below, at and just past a block's output cells, for every kind
of boundary and cell, eager and as a graph."""
import numpy as np
import pytest
import torch

from paper_2404_01035_amd import abi, inputs

pytestmark = pytest.mark.gpu


def _instance(n, N, K, precision, bc, delta=0.0, potential="well", ext=False, seed=5):
    p, _, _ = inputs.random_instance(np.random.default_rng(seed), 16, 16, N, K, nuclei=1)
    p = p.copy(n=(n[0], n[1], 1), precision=precision, potential=potential)
    p.bc = bc + (0,)
    p.G, p.V, p.y0 = 1e-3, 0.01, 3.0
    if delta:
        p.delta[:, :] = delta * (1.0 - np.eye(3))
    if ext:
        p.Bt[:N, :K - 1] = 0.05
        p.Ct[:N] = 0.02
    p.dt = 0.2 * inputs.dt_limit(p)
    phi, mu = inputs.random_multiphase(p, seed)
    return p, phi, mu


def _run(p, phi, mu, nsteps, strips, graph=0, reps=1):
    from paper_2404_01035_amd.solver import Solver

    s = Solver(p)
    if strips:
        s.set_tile(256, 7, 1)
    s.set_graph(graph)
    s.load(phi, mu, step=11)
    for _ in range(reps):
        s.step(nsteps)
    torch.cuda.synchronize()
    out = s.current().clone()
    where = abi.mp_current(s.st)
    s.close()
    return out, where


CASES = [
    ((1, 1), 2, 2, "f64", (0, 0), {}), ((5, 3), 3, 3, "f64", (1, 0), {}), ((1, 40), 3, 2, "f32", (1, 1), {}),
    ((64, 64), 2, 2, "f64", (0, 0), {}), ((48, 36), 3, 3, "f64", (0, 1), {"delta": 0.03}),
    ((65, 33), 3, 3, "f32", (1, 1), {"delta": 0.02, "potential": "obstacle"}),
    ((300, 70), 2, 3, "f64", (0, 1), {"potential": "obstacle"}), ((257, 129), 3, 3, "f32", (0, 0), {}),
    ((31, 95), 3, 3, "f64", (1, 0), {"ext": True}), ((33, 17), 2, 2, "f32", (1, 1), {"ext": True, "delta": 0.02}),
    ((40, 41), 3, 3, "f64", (0, 1), {"potential": "obstacle_active", "delta": 0.02}),
    ((512, 256), 3, 3, "f32", (0, 1), {}), ((256, 256), 2, 2, "f64", (1, 0), {}),
]


@pytest.mark.parametrize("n,N,K,precision,bc,kw", CASES)
def test_tiles_step_the_strips_bits(n, N, K, precision, bc, kw):
    p, phi, mu = _instance(n, N, K, precision, bc, **kw)
    for nsteps in (3, 8, 25):
        tiles, strips = (_run(p, phi, mu, nsteps, s) for s in (False, True))
        assert tiles[1] == strips[1]
        assert torch.equal(tiles[0], strips[0]), nsteps


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_tiles_in_a_replayed_graph(precision):
    p, phi, mu = _instance((70, 45), 3, 3, precision, (0, 1))
    tiles, strips = (_run(p, phi, mu, 10, s, graph=g, reps=4) for s, g in ((False, 10), (True, 0)))
    assert tiles[1] == strips[1]
    assert torch.equal(tiles[0], strips[0])


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_adjoint_over_states_stored_by_tiles(precision):
    """The recomputation's tiles also store the states between their steps."""
    from paper_2404_01035_amd.solver import Solver

    p, phi, mu = _instance((60, 41), 3, 3, precision, (0, 1))
    p.G = p.V = 0.0
    rng = np.random.default_rng(1)
    lam = torch.from_numpy(rng.normal(size=(p.nfields,) + tuple(p.spatial))).cuda()
    got = []
    for strips in (False, True):
        s = Solver(p)
        if strips:
            s.set_tile(256, 7, 1)
        s.load(phi, mu)
        ckpt = s.checkpoint_buffer(23, 11)
        s.step_ckpt(23, 11, ckpt)
        lam0, g = s.adjoint(lam, ckpt, 23, 11, 0)
        got.append((lam0.clone(), g))
        s.close()
    assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
