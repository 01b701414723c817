"""Which calls the register windows and the row pipeline take: calls of few sweeps
on grids too large for them, where they were measured slower than the persistent
kernel or the half-sweeps, go there; the library's own rule, on the CPU."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2607_01735_amd", "librbgs.so")
F64, F32 = 8, 4


@pytest.fixture(scope="module")
def takes():
    lib = ctypes.CDLL(LIB)
    fn = lib["_ZN4rbgs12window_takesEimibb"]
    fn.restype = ctypes.c_bool

    def call(n, elem, sweeps, in_place=False, sor=False):
        return fn(n, ctypes.c_size_t(elem), sweeps, ctypes.c_bool(in_place), ctypes.c_bool(sor))

    return call


@pytest.mark.parametrize("n,elem,sweeps", [
    (16383, F64, 8), (16383, F64, 9), (16383, F64, 20), (24575, F64, 9), (24575, F64, 30),
    (10001, F32, 8), (10001, F32, 14), (12287, F32, 8), (12287, F32, 14), (12287, F32, 20),
    (16383, F32, 9), (16383, F32, 24), (24575, F32, 20), (32767, F32, 12),
    (4095, F64, 1), (8191, F64, 40), (12287, F32, 30),
])
def test_slower_calls_go_elsewhere(takes, n, elem, sweeps):
    assert not takes(n, elem, sweeps)
    assert not takes(n, elem, sweeps, in_place=True)


@pytest.mark.parametrize("n,elem,sweeps,sor", [
    (8191, F64, 2, False), (12287, F64, 2, False), (7001, F32, 2, False), (12287, F32, 2, False),
    (4095, F64, 2, True), (2047, F64, 2, True), (12287, F64, 30, False), (5001, F32, 14, False),
    (8191, F32, 14, False), (8191, F32, 16, False), (12287, F32, 16, False), (9001, F32, 50, False),
    (255, F64, 1, False), (255, F32, 1, False),
])
def test_slower_in_place(takes, n, elem, sweeps, sor):
    """Two-buffer passes that have to end where they start: an odd number takes
    one more, shallower; two sweeps take two passes of one."""
    assert not takes(n, elem, sweeps, in_place=True, sor=sor)


@pytest.mark.parametrize("n,elem,sweeps,in_place", [
    (63, F64, 10, True), (255, F64, 1000, True), (2300, F64, 50, True), (8000, F64, 1000, True),
    (8191, F64, 30, True), (12287, F64, 20, False), (24575, F64, 7, True), (1000, F32, 200, True),
    (8191, F32, 100, False), (8191, F32, 30, True), (4095, F32, 14, True), (12287, F32, 12, True),
    (12287, F32, 24, False), (12287, F64, 16, True), (7001, F32, 16, True), (32767, F32, 7, True), (4095, F64, 2, True), (4095, F32, 2, True),
])
def test_faster_calls_stay(takes, n, elem, sweeps, in_place):
    assert takes(n, elem, sweeps, in_place=in_place)


@pytest.mark.parametrize("elem", [F64, F32])
def test_in_place_is_the_narrower_rule(takes, elem):
    for n in (1, 64, 512, 1600, 2301, 4300, 4301, 5500, 5501, 8000, 8001, 8200, 8201, 9200, 9201,
              10000, 10001, 12000, 12001, 12500, 12501, 15500, 15501, 65533):
        for sweeps in list(range(1, 64)) + [100, 1000, 2 ** 31 - 1]:
            for sor in (False, True):
                assert takes(n, elem, sweeps, False, sor) or not takes(n, elem, sweeps, True, sor)
