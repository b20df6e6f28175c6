"""The tuner against the default tile: it is one of the candidates, stays set
where it wins, and comes back from the cache whatever tile was set before."""
import pytest

from paper_2404_01035_amd import abi, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision", [((64, 64), "f64"), ((128, 96), "f32")])
def test_small_grids_keep_the_default(n, precision, tmp_path):
    from paper_2404_01035_amd.solver import Solver

    p, phi, mu = inputs.config_c2(n=(n[0], n[1], 1), precision=precision)
    cache = str(tmp_path / "tiles.json")
    for source in ("timed", "cache"):
        s = Solver(p)
        try:
            s.load(phi, mu)
            launches = abi.mp_get_launches(s.st, 100)
            assert launches[3] > 0  # the tile kernel
            s.set_tile(64, 8, 1)
            r = s.autotune(reps=5, cache=cache)
            # several steps per launch: 2 to 4 times faster than any set tile here
            assert r["source"] == source and r["default"] and r["fuse"] == 2
            assert abi.mp_get_launches(s.st, 100) == launches
            assert min(r["ms"], key=r["ms"].get) == "0,0,0,2"
        finally:
            s.close()


def test_a_failed_tuning_leaves_the_tile(tmp_path):
    from paper_2404_01035_amd.solver import Solver

    s = Solver(inputs.dendrite_params(n=(40, 24, 20)))
    try:
        before = abi.mp_get_tile(s.st), abi.mp_get_launches(s.st, 1)
        with pytest.raises(abi.MPError):
            abi.mp_tune(s.st, [(256, 4, 1, 2), (100, 4, 1, 1)], 2, s.stream())  # none is valid in 3D
        assert (abi.mp_get_tile(s.st), abi.mp_get_launches(s.st, 1)) == before
        with pytest.raises(abi.MPError):
            abi.mp_tune(s.st, [(512, 4, 2, 1)], 2, s.stream())
        assert (abi.mp_get_tile(s.st), abi.mp_get_launches(s.st, 1)) == before
    finally:
        s.close()
