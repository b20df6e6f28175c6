"""What mp_step launches (mp_get_launches), host side: no GPU needed."""
import ctypes as C

import numpy as np
import pytest

from paper_2404_01035_amd import abi, inputs


@pytest.fixture
def state():
    made = []

    def make(p):
        made.append(abi.mp_create(p))
        return made[-1]

    yield make
    for st in made:
        abi.mp_destroy(st)


def test_the_3d_default_is_the_tile_that_is_launched(state):
    st = state(inputs.dendrite_params(n=(512, 512, 512)))
    assert abi.mp_get_tile(st)[:2] == (256, 64)
    assert abi.mp_get_launches(st, 4) == (4, 256, 64, 0)


def test_a_segment_alone_leaves_the_3d_tile(state):
    st = state(inputs.dendrite_params(n=(96, 80, 70)))
    bx = abi.mp_get_launches(st, 1)[1]
    abi.mp_set_tile(st, 0, 16, 0)
    assert abi.mp_get_launches(st, 1) == (1, bx, 16, 0)
    abi.mp_set_tile(st, 512, 0, 0)
    assert abi.mp_get_launches(st, 1) == (1, 512, 16, 0)


def test_launches_of_2d_grids(state):
    p = inputs.eutectic_params(n=(4096, 4096, 1))
    assert abi.mp_get_launches(state(p), 9) == (5, 256, 31, 0)
    st = state(inputs.config_c1()[0])
    count, bx, seg, region = abi.mp_get_launches(st, 100)
    assert region in (16, 24, 32) and bx == region * region and seg == 0
    assert count < 50 and count % 2 == 0  # as many launches as the strips' 50, modulo 2
    abi.mp_set_tile(st, 256, 0, 0)
    count, bx, seg, region = abi.mp_get_launches(st, 100)
    assert (count, bx, region) == (50, 256, 0) and 1 <= seg < 31


def test_argument_errors(state):
    st = state(inputs.config_c1()[0])
    L = abi.lib()
    assert L.mp_get_launches(None, 1, None, None, None, None) == abi.MP_E_NULLPTR
    assert L.mp_get_launches(st, 0, None, None, None, None) == abi.MP_E_PARAM
    n = C.c_int64()
    assert L.mp_get_launches(st, 1, C.byref(n), None, None, None) == abi.MP_OK and n.value == 1


def test_3d_segments_where_a_simd_holds_one_wave(state):
    # FP64, anisotropic, general, five fields: the second block of a CU waits for the
    # first, so 256^3 keeps the longest segments and 96 x 80 x 70 (30 tiles) takes
    # segments that make one round of at most 256 blocks
    p, _, _ = inputs.random_instance(np.random.default_rng(7), 16, 16, 3, 3, nuclei=1)
    p.delta[:, :] = 0.02 * (1.0 - np.eye(3))
    p.Bt[:3, :2] = 0.05

    def seg(n):
        q = p.copy(n=n, dim=3, precision="f64")
        q.dt = 0.2 * inputs.dt_limit(q)
        return abi.mp_get_launches(state(q), 1)[2]

    assert seg((256, 256, 256)) == 64
    assert 30 * -(-70 // seg((96, 80, 70))) <= 256


@pytest.mark.parametrize("members,side,precision,segs", [
    # measured within 7 % of the best of 2 .. 32 rows (us per step, 32 rows / best)
    (24, (128, 400), "f64", (6, 8, 12, 16)),      # 33.9 / 21.9
    (8, (64, 1024), "f64", (8, 12, 16, 28)),      # 50.0 / 43.4
    (64, (64, 1024), "f64", (20, 24, 28, 32)),    # 217 / 217
    (24, (128, 400), "f32", (4, 6, 8)),           # 32.3 / 14.6 (the mean strip's model)
    (64, (64, 1024), "f32", (24, 28, 32)),        # 127 / 124
])
def test_batch_segments_follow_the_deal(state, members, side, precision, segs):
    rng = np.random.default_rng({(24, 128): 8, (8, 64): 6, (64, 64): 7}[members, side[0]])
    ps = []
    for i in range(members):
        nx, ny = (int(rng.integers(side[0], side[1] + 1)) for _ in range(2))
        N, K = ((2, 2), (3, 3), (3, 2))[i % 3]
        p, _, _ = inputs.random_instance(np.random.default_rng(7), 16, 16, N, K, nuclei=1)
        p = p.copy(n=(nx, ny, 1), precision=precision)
        p.dt = 0.2 * inputs.dt_limit(p)
        ps.append(p)
    st = abi.mp_create_batch(ps)
    try:
        assert abi.mp_get_launches(st, 4)[2] in segs
        abi.mp_set_tile(st, 0, 11, 0)
        assert abi.mp_get_launches(st, 4) == (2, 256, 11, 0)
    finally:
        abi.mp_destroy(st)


@pytest.mark.parametrize("make", [
    lambda: abi.mp_create(inputs.config_c1()[0]),
    lambda: abi.mp_create(inputs.eutectic_params(n=(1024, 768, 1), precision="f32")),
    lambda: abi.mp_create(inputs.dendrite_params(n=(96, 80, 70))),
    lambda: abi.mp_create_batch([m[0] for m in inputs.config_c4(ninst=3, side=(64, 90))]),
])
def test_all_zero_goes_back_to_the_default_tile(make):
    st = make()
    try:
        tile, launches = abi.mp_get_tile(st), abi.mp_get_launches(st, 40)
        abi.mp_set_tile(st, 0, 9, 1)
        assert abi.mp_get_launches(st, 40) != launches
        abi.mp_set_tile(st, 0, 0, 0)
        assert (abi.mp_get_tile(st), abi.mp_get_launches(st, 40)) == (tile, launches)
    finally:
        abi.mp_destroy(st)


def test_tuned_tiles_belong_to_one_build(monkeypatch):
    from paper_2404_01035_amd import autotune

    p = inputs.config_c1()[0]
    a = autotune.signature([p], "dev")
    monkeypatch.setattr(autotune, "library_id", lambda: "another build")
    assert autotune.signature([p], "dev") != a


@pytest.mark.parametrize("n,N,K,precision,aniso,ext,tiles", [
    # measured with 24 steps, us per step of the tile kernel / the strips
    ((512, 512), 3, 2, "f64", True, False, False),   # 15.6 / 10.7
    ((400, 300), 3, 3, "f64", True, True, False),    # 15.1 / 11.5
    ((768, 640), 3, 3, "f32", True, False, False),   # 13.9 / 11.3
    ((768, 640), 2, 3, "f32", False, True, False),   # 7.6 / 6.4
    ((512, 512), 3, 3, "f32", True, False, True),    # 9.2 / 9.9
    ((64, 64), 3, 3, "f64", True, True, True),       # 4.4 / 6.9
    ((512, 512), 2, 2, "f64", False, False, True),   # 4.1 / 4.5
])
def test_tiles_only_where_they_are_faster(state, n, N, K, precision, aniso, ext, tiles):
    p, _, _ = inputs.random_instance(np.random.default_rng(7), 16, 16, N, K, nuclei=1)
    p = p.copy(n=(n[0], n[1], 1), precision=precision)
    if aniso:
        p.delta[:, :] = 0.02 * (1.0 - np.eye(3))
    if ext:
        p.Bt[:N, :K - 1] = 0.05
    p.dt = 0.2 * inputs.dt_limit(p)
    assert (abi.mp_get_launches(state(p), 24)[3] > 0) == tiles
