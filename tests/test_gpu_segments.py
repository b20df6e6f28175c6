"""Segments picked by a launch (no tile set) against the default's full length:
the same bits, on grids that leave most of the GPU idle, on either side of one
strip, and with the anti-trapping current, the extended model, 3D and batches."""
import numpy as np
import pytest
import torch

from paper_2404_01035_amd import abi, inputs

pytestmark = pytest.mark.gpu


def _instance(n, N, K, precision, seed=3, **kw):
    p, _, _ = inputs.random_instance(np.random.default_rng(seed), 16, 16, N, K, nuclei=1)
    p = p.copy(n=tuple(n), dim=3 if n[2] > 1 else 2, precision=precision)
    for k, v in kw.items():
        setattr(p, k, v)
    p.dt = 0.2 * inputs.dt_limit(p)
    phi, mu = inputs.random_multiphase(p, seed)
    return p, phi, mu


def _run(p, phi, mu, nsteps, seg, at):
    from paper_2404_01035_amd.solver import Solver

    s = Solver(p)
    if seg:
        s.set_tile(0, seg, 0)
    s.load(phi, mu)
    if at:
        s.set_antitrapping(at)
    s.step(nsteps)
    out = s.current().clone()
    torch.cuda.synchronize()
    s.close()
    return out


@pytest.mark.parametrize("n,precision,bc,at,ext", [
    ((60, 33, 1), "f64", (0, 1, 0), 0, False), ((61, 64, 1), "f32", (1, 0, 0), 0, False),
    ((300, 70, 1), "f64", (1, 1, 0), 1, False), ((127, 90, 1), "f32", (0, 0, 0), 2, False),
    ((97, 50, 1), "f64", (0, 1, 0), 0, True), ((64, 9, 40), "f32", (1, 1, 1), 0, False),
    ((65, 13, 70), "f64", (0, 1, 0), 1, False), ((30, 21, 67), "f32", (1, 0, 1), 1, True),
])
def test_picked_segments_change_no_bits(n, precision, bc, at, ext):
    kw = {"bc": bc}
    if ext:
        kw["tau_ab"] = 1.0 - np.eye(3)
    p, phi, mu = _instance(n, 3, 3, precision, **kw)
    default = abi.mp_create(p)
    seg = abi.mp_get_tile(default)[1]
    abi.mp_destroy(default)
    picked, full = (_run(p, phi, mu, 5, s, at) for s in (0, seg))
    assert torch.equal(picked, full)


@pytest.mark.parametrize("at", [False, True])
def test_picked_batch_segments_change_no_bits(at):
    from paper_2404_01035_amd.solver import BatchSolver

    made = [_instance((nx, ny, 1), N, K, "f32", seed=i) for i, (nx, ny, N, K) in
            enumerate([(64, 300, 2, 2), (130, 35, 3, 3), (61, 7, 3, 2)])]
    out = []
    for seg in (0, 32):
        b = BatchSolver([m[0] for m in made])
        if seg:
            b.set_tile(seg)
        for i, (_, phi, mu) in enumerate(made):
            b.load(i, phi, mu)
        b.start(0)
        b.set_antitrapping(at)
        b.step(5)
        out.append([b.fields(i) for i in range(len(made))])
        b.close()
    for (f0, u0), (f1, u1) in zip(*out):
        assert np.array_equal(f0, f1) and np.array_equal(u0, u1)
