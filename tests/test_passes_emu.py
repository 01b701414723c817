"""The fused passes' kernels and launchers, run on the CPU, against the oracle.

Register windows, the row pipeline (the tile pipeline with one column a lane), the
multigrid legs and the 9-point passes are compiled unchanged for the host
(`tests/emu/passes_emu.cpp`: a wave's 64 lanes as fibers, every array a heap block of
exactly the library's size, all of it NaN until it is written).  AddressSanitizer
reports any access outside an array; the results are the oracle's bit for bit.  Sizes:
a single point, grids smaller than a tile, and ones with tiles that touch no edge,
odd and even.  The ring of f is NaN: it must not be used.
"""
import concurrent.futures as cf
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "emu", "passes_emu.cpp")
INCLUDES = [os.path.join(ROOT, "tests", "emu"), os.path.join(ROOT, "paper_2607_01735_amd", "csrc"),
            os.path.join(ROOT, "include")]
KINDS = {"windows": [], "pipeline": ["-DEMU_PIPELINE"], "mc9": ["-DEMU_MC9"], "legs": ["-DEMU_LEGS"]}

pytestmark = [pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++"), pytest.mark.slow]


@pytest.fixture(scope="module")
def emulators(tmp_path_factory):
    out = tmp_path_factory.mktemp("passes_emu")

    def build(kind):
        exe = out / kind
        # no _FORTIFY_SOURCE: its longjmp check rejects the jumps between fiber stacks
        cmd = (["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-U_FORTIFY_SOURCE",
                "-fsanitize=address", "-Wno-attributes"] + KINDS[kind] +
               [f"-I{d}" for d in INCLUDES] + [SRC, "-o", str(exe)])
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-3000:]
        return kind, exe

    with cf.ThreadPoolExecutor(len(KINDS)) as ex:
        return dict(ex.map(build, KINDS))


def run(exe, tmp_path, n, sweeps, fuse=0, omega=1.0, dtype=np.float64):
    """(result, the double that follows it, start, f with a zero ring, h)"""
    h = W.spacing(n)
    u = W.random_ring(n, seed=n)
    u[1:n + 1, 1:n + 1] = W.uniform_rhs(n, seed=n + 1)[1:n + 1, 1:n + 1]
    u = np.ascontiguousarray(u.astype(dtype))
    f = np.full_like(u, np.nan)
    f[1:n + 1, 1:n + 1] = W.uniform_rhs(n, seed=n + 2)[1:n + 1, 1:n + 1]
    fin, fout = tmp_path / "in.bin", tmp_path / "out.bin"
    fin.write_bytes(u.tobytes() + f.tobytes())
    res = subprocess.run([str(exe), np.dtype(dtype).name, str(n), str(sweeps), str(fuse), repr(omega),
                          repr(h), str(fin), str(fout)], capture_output=True, text=True, timeout=600,
                         env=dict(os.environ,
                                  ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0"))
    assert res.returncode == 0, (res.stdout + res.stderr)[-4000:]
    raw = fout.read_bytes()
    got = np.frombuffer(raw[:-8], dtype=dtype).reshape(u.shape)
    return got, np.frombuffer(raw[-8:], dtype=np.float64)[0], u, np.nan_to_num(f), h


@pytest.mark.parametrize("kind,n,sweeps,fuse,omega,dtype", [
    ("windows", 1, 3, 2, 1.0, np.float64), ("windows", 7, 9, 5, 1.0, np.float64),
    ("windows", 230, 9, 5, 1.0, np.float64), ("windows", 131, 7, 4, 1.5, np.float64),
    ("windows", 2, 6, 6, 1.0, np.float32), ("windows", 229, 11, 6, 1.0, np.float32),
    ("pipeline", 7, 12, 7, 1.0, np.float64), ("pipeline", 64, 9, 5, 1.0, np.float64),
    ("pipeline", 240, 7, 7, 1.0, np.float64), ("pipeline", 231, 8, 4, 1.5, np.float64),
])
def test_sweeps(oracle, emulators, tmp_path, kind, n, sweeps, fuse, omega, dtype):
    got, _, ref, f, h = run(emulators[kind], tmp_path, n, sweeps, fuse, omega, dtype)
    if omega == 1.0:
        oracle.sweep(ref, f, h, sweeps)
    else:
        oracle.sor_sweep(ref, f, h, omega, sweeps)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("n,sweeps,fuse", [(1, 3, 3), (2, 3, 2), (62, 4, 3), (141, 3, 3), (140, 2, 1)])
def test_nine_point(oracle, emulators, tmp_path, n, sweeps, fuse):
    got, _, u, f, h = run(emulators["mc9"], tmp_path, n, sweeps, fuse)
    assert np.array_equal(got, oracle.mc9_sweep(u, f, h, sweeps))


@pytest.mark.parametrize("n,nu", [(3, 1), (5, 2), (63, 2), (301, 1), (511, 2)])
def test_multigrid_legs(oracle, emulators, tmp_path, n, nu):
    """A cycle of two levels; the norm's sum of n^2 squares in another order."""
    got, squares, ref, f, h = run(emulators["legs"], tmp_path, n, nu)
    oracle.mg_solve(ref, f, h, nu, nu, 1, -1.0, max_levels=2, coarse_sweeps=3)
    assert np.array_equal(got, ref)
    norm, _ = oracle.residual(ref, f, h)
    assert abs(np.sqrt(squares) - norm) <= n * n * 2.0 ** -53 * norm
