"""The strips' marches at their shortest and at odd and even lengths: segments of
1 to 4 rows, grids of 1 to 7 rows, one and two steps per launch, with the
anti-trapping current and the extended model, against the oracle (three steps:
FP64 rounding stays below 1e-12, FP32 below 1e-5); and batches whose strips do
and do not hold a mirrored column, against single grids to the bit."""
import numpy as np
import pytest

from oracle import gp
from paper_2404_01035_amd import inputs

pytestmark = pytest.mark.gpu


def _instance(n, N, K, precision, bc, ext=False):
    p, _, _ = inputs.random_instance(np.random.default_rng(11), 16, 16, N, K, nuclei=1)
    p = p.copy(n=n, dim=2, precision=precision)
    p.bc = bc
    p.G, p.V, p.y0 = 1e-3, 0.01, 3.0
    if ext:
        p.Bt[:N, :K - 1] = 0.05
    p.dt = 0.2 * inputs.dt_limit(p)
    phi, mu = inputs.random_multiphase(p, 5)
    if precision == "f32":
        phi, mu = phi.astype(np.float32).astype(float), mu.astype(np.float32).astype(float)
    return p, phi, mu


@pytest.mark.parametrize("ny", [1, 2, 3, 4, 7])
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 1, 0), (0, 1, 0)])
@pytest.mark.parametrize("precision,fuse,at,ext", [
    ("f64", 1, 0, False), ("f32", 2, 0, False), ("f64", 2, 0, True), ("f64", 1, 1, False), ("f32", 1, 1, True),
])
def test_short_marches_against_the_oracle(ny, bc, precision, fuse, at, ext):
    from paper_2404_01035_amd.solver import Solver

    p, phi, mu = _instance((63, ny, 1), 3, 3, precision, bc, ext)
    want = phi, mu
    for i in range(3):
        want = (gp.step_antitrapping if at else gp.step)(*want, 5 + i, p)
    tol = 1e-12 if precision == "f64" else 1e-5
    for seg in (1, 2, 3, 4):
        s = Solver(p)
        s.set_tile(256, seg, 1)
        s.set_fusion(fuse)
        s.set_antitrapping(at)
        s.load(phi, mu, 5)
        s.step(3)
        got = s.fields()
        s.close()
        for a, b in zip(got, want):
            assert np.max(np.abs(a - b)) <= tol, seg


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("ext", [False, True])
def test_batches_with_and_without_mirrored_columns(precision, ext):
    from paper_2404_01035_amd.solver import BatchSolver, Solver

    insts = [_instance((nx, ny, 1), N, K, precision, bc, ext) for nx, ny, N, K, bc in (
        (64, 33, 3, 3, (0, 1, 0)), (64, 33, 3, 3, (1, 0, 0)), (60, 5, 2, 2, (1, 1, 0)), (119, 9, 2, 3, (0, 0, 0)),
        (121, 9, 3, 2, (1, 0, 0)), (181, 7, 2, 2, (0, 1, 0)), (7, 3, 2, 2, (0, 0, 0)))]
    b = BatchSolver([i[0] for i in insts])
    for i, (_, phi, mu) in enumerate(insts):
        b.load(i, phi, mu)
    b.start(0)
    b.step(5)
    for i, (p, phi, mu) in enumerate(insts):
        s = Solver(p)
        s.load(phi, mu)
        s.step(5)
        for a, w in zip(b.fields(i), s.fields()):
            assert np.array_equal(a, w), i
        s.close()
    b.close()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("vec", [1, 2])
@pytest.mark.parametrize("ext,at", [(False, 0), (True, 0), (False, 1), (True, 1)])
def test_batches_with_rows_that_fit_a_wave(precision, vec, ext, at):
    """Periodic rows of exactly 64 cells per lane held, one column either side, and the same width with mirrors."""
    from paper_2404_01035_amd.solver import BatchSolver, Solver

    insts = [_instance((nx, ny, 1), N, K, precision, bc, ext) for nx, ny, N, K, bc in (
        (64, 33, 3, 3, (0, 1, 0)), (64, 5, 2, 2, (0, 0, 0)), (64, 9, 2, 2, (1, 0, 0)), (128, 9, 3, 2, (0, 0, 0)),
        (128, 4, 2, 3, (0, 1, 0)), (62, 9, 2, 2, (0, 0, 0)), (66, 9, 3, 3, (0, 0, 0)), (63, 3, 2, 2, (0, 0, 0)),
        (130, 3, 2, 2, (0, 0, 0)), (192, 3, 2, 2, (0, 0, 0)))]
    b = BatchSolver([i[0] for i in insts])
    b.set_tile(32, vec)
    for i, (_, phi, mu) in enumerate(insts):
        b.load(i, phi, mu)
    b.start(0)
    b.set_antitrapping(at)
    b.step(5)
    for i, (p, phi, mu) in enumerate(insts):
        s = Solver(p)
        s.load(phi, mu)
        s.set_antitrapping(at)
        s.step(5)
        for a, w in zip(b.fields(i), s.fields()):
            assert np.array_equal(a, w), i
        s.close()
    b.close()
