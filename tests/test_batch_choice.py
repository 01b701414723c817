"""Which batches the register windows take: the library's own rule, on the CPU.
Batches of several large FP64 grids, whose tiles fill the chip, go to the persistent
kernel in long calls, where it was measured faster."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2607_01735_amd", "librbgs.so")
F64, F32 = 8, 4


@pytest.fixture(scope="module")
def pay():
    fn = ctypes.CDLL(LIB)["_ZN4rbgs17batch_windows_payEiPKimi"]
    fn.restype = ctypes.c_bool

    def call(sizes, elem, sweeps):
        return fn(len(sizes), (ctypes.c_int * len(sizes))(*sizes), ctypes.c_size_t(elem), sweeps)

    return call


@pytest.mark.parametrize("sizes,elem,sweeps", [
    ([4095] * 8, F64, 20), ([4095] * 8, F64, 100), ([4095] * 4, F64, 100), ([3000] * 8, F64, 100),
    ([2300] * 16, F64, 100), ([2300] * 12, F64, 50), ([2300] * 14, F64, 30), ([3500] * 16, F64, 10),
    ([2047] * 16, F64, 30), ([1600] * 32, F64, 50), ([1800] * 48, F64, 100),
    ([4095] * 3 + [1023] * 16, F64, 100), ([4095] * 4 + [255] * 128, F64, 100),
    ([8191] * 3, F32, 14), ([10000] * 3, F32, 14), ([4096], F64, 4), ([10001], F32, 4),
])
def test_persistent_is_faster(pay, sizes, elem, sweeps):
    assert not pay(sizes, elem, sweeps)


@pytest.mark.parametrize("sizes,elem,sweeps", [
    ([4095] * 8, F64, 8), ([4095] * 4, F64, 20), ([4095] * 2, F64, 100), ([4095], F64, 1000),
    ([3000] * 4, F64, 100), ([2300] * 8, F64, 100), ([2300] * 16, F64, 8), ([1500] * 32, F64, 100),
    ([1023] * 64, F64, 100), ([63] * 4096, F64, 100), ([4095] * 4 + [255] * 128, F64, 20),
    ([1800] * 48, F64, 30), ([8191] * 4, F32, 100), ([4095] * 16, F32, 20), ([1023] * 256, F32, 20),
    ([63, 127, 255, 511, 1023] * 100, F32, 100), ([1], F64, 2 ** 31 - 1), ([1], F32, 1),
])
def test_windows_are_faster(pay, sizes, elem, sweeps):
    assert pay(sizes, elem, sweeps)
