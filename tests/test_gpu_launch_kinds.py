"""Every kind of launch that mp_step picks without a set tile, checked to be the
one that ran (mp_get_launches), against the strips at a set tile: the same bits
in the same buffer.  The tile kernel at each region size, precision, face and
cell kind and field count, regions of up to 144 KiB of LDS among them; the
strips' picked segments."""
import numpy as np
import pytest
import torch

from paper_2404_01035_amd import abi, inputs

pytestmark = pytest.mark.gpu

GRIDS = [(5, 3), (31, 33), (64, 70), (97, 50), (129, 40), (200, 131), (257, 129), (300, 200), (512, 100), (33, 799), (61, 799)]
STEPS = (10, 9, 13, 7, 12, 25, 5)


def _instance(n, N, K, precision, bc=(0, 1), aniso=False, ext=False):
    p, _, _ = inputs.random_instance(np.random.default_rng(7), 16, 16, N, K, nuclei=1)
    p = p.copy(n=(n[0], n[1], 1), precision=precision)
    p.bc = bc + (0,)
    p.G, p.V, p.y0 = 1e-3, 0.01, 3.0
    if aniso:
        p.delta[:, :] = 0.02 * (1.0 - np.eye(3))
    if ext:
        p.Bt[:N, :K - 1] = 0.05
    p.dt = 0.2 * inputs.dt_limit(p)
    return p


def _run(p, nsteps, tile):
    from paper_2404_01035_amd.solver import Solver

    phi, mu = inputs.random_multiphase(p, 3)
    s = Solver(p)
    if tile:
        s.set_tile(*tile)
    launches = abi.mp_get_launches(s.st, nsteps)
    s.load(phi, mu, step=11)
    s.step(nsteps)
    torch.cuda.synchronize()
    out = s.current().clone(), abi.mp_current(s.st)
    s.close()
    return out, launches


def _pick(make, region):
    """The first grid and step count of the lists that take regions of this size."""
    for n in GRIDS:
        st = abi.mp_create(make(n))
        try:
            for nsteps in STEPS:
                if abi.mp_get_launches(st, nsteps)[3] == region:
                    return n, nsteps
        finally:
            abi.mp_destroy(st)
    return None


@pytest.mark.parametrize("region", [16, 24, 32])
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("aniso", [False, True])
@pytest.mark.parametrize("ext", [False, True])
def test_tile_regions(region, precision, aniso, ext):
    for N, K in ((2, 2), (3, 2), (2, 3), (3, 3)):
        def make(n):
            return _instance(n, N, K, precision, (N & 1, K & 1), aniso, ext)

        picked = _pick(make, region)
        if picked is None:  # slower than smaller regions at any size: FP64, anisotropic, five fields
            assert (precision, aniso, ext, N, K, region) == ("f64", True, False, 3, 3, 32)
            continue
        n, nsteps = picked
        print(f"{precision} N={N} K={K} aniso={aniso} ext={ext}: {nsteps} steps of {n} on {region}^2", flush=True)
        tiles, launches = _run(make(n), nsteps, None)
        strips, other = _run(make(n), nsteps, (256, 7, 1))
        assert launches[3] == region and other[3] == 0
        assert tiles[1] == strips[1]
        assert torch.equal(tiles[0], strips[0]), (n, nsteps, N, K)


@pytest.mark.parametrize("n,precision,bc,ext", [
    ((60, 33), "f64", (0, 1), False), ((61, 64), "f32", (1, 0), False), ((97, 50), "f64", (0, 1), True),
    ((700, 301), "f32", (1, 1), True), ((1024, 90), "f64", (0, 0), False),
])
@pytest.mark.parametrize("nsteps", [1, 2])
def test_picked_strip_segments(n, precision, bc, ext, nsteps):
    p = _instance(n, 3, 3, precision, bc, ext=ext)
    full = 31 if precision == "f64" else 14
    picked, launches = _run(p, nsteps, None)
    default, _ = _run(p, nsteps, (0, full, 0))
    assert launches[3] == 0 and 1 <= launches[2] < full
    assert picked[1] == default[1] and torch.equal(picked[0], default[0])
