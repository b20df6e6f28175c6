"""3D tiles at the sizes where they can go wrong: one cell below, at and past a
tile in x and y, one plane to a few past a segment, every boundary, isotropic
(two planes in LDS) and anisotropic (rings of four and three), against the
oracle.  Three steps: FP64 rounding stays below 1e-12, FP32 below 1e-5."""
import numpy as np
import pytest

from oracle import gp
from paper_2404_01035_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc,N,K,delta,ext,precision", [
    ((31, 7, 1), (0, 0, 0), 2, 2, 0.0, False, "f64"), ((32, 8, 2), (1, 0, 1), 3, 3, 0.0, False, "f64"),
    ((33, 9, 3), (0, 1, 0), 3, 3, 0.0, False, "f32"), ((65, 17, 6), (1, 1, 1), 2, 3, 0.0, True, "f64"),
    ((1, 1, 4), (0, 1, 0), 3, 2, 0.0, False, "f64"), ((31, 9, 5), (1, 0, 0), 2, 2, 0.03, False, "f64"),
    ((32, 8, 1), (0, 1, 1), 3, 3, 0.02, False, "f32"), ((64, 7, 4), (1, 1, 0), 3, 3, 0.02, False, "f64"),
    ((3, 2, 2), (0, 0, 0), 2, 2, 0.03, False, "f64"), ((33, 16, 5), (0, 0, 1), 2, 2, 0.02, True, "f32"),
])
@pytest.mark.parametrize("seg", [0, 2])
def test_tiles_against_the_oracle(n, bc, N, K, delta, ext, precision, seg):
    from paper_2404_01035_amd.solver import Solver

    p, _, _ = inputs.random_instance(np.random.default_rng(7), 16, 16, N, K, nuclei=1)
    p = p.copy(n=n, dim=3, precision=precision)
    p.bc = bc
    if delta:
        p.delta[:, :] = delta * (1.0 - np.eye(3))
    if ext:
        p.Bt[:N, :K - 1] = 0.05
    p.G, p.V, p.y0 = 1e-3, 0.01, 3.0
    p.dt = 0.2 * inputs.dt_limit(p)
    phi, mu = inputs.random_multiphase(p, 3)
    if precision == "f32":
        phi, mu = phi.astype(np.float32).astype(float), mu.astype(np.float32).astype(float)
    s = Solver(p)
    if seg:
        s.set_tile(256, seg, 0)
    s.load(phi, mu, step=5)
    s.step(3)
    got = s.fields()
    s.close()
    want = gp.run(phi, mu, 5, 3, p)
    tol = 1e-12 if precision == "f64" else 1e-5
    for a, b in zip(got, want):
        assert np.max(np.abs(a - b)) <= tol
