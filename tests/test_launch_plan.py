"""What mp_step launches (mp_get_launches), host side: no GPU needed."""
import ctypes as C

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
