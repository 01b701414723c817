"""The register windows (automatic kernel) against the plain half-sweeps, bit
for bit, and those against the oracle on the small sizes: sizes on both sides
of a window's columns and strips and of every switch of shape, odd and even n,
every depth, odd and even launch counts, SOR, rounds of a solve, refinement, a
ring of f that must not be read, and the split layout."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402

F64, F32 = torch.float64, torch.float32


def grid(n, seed, ld, dtype):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    u = torch.rand((n + 2, ld), generator=g, device="cuda:0", dtype=F64).mul_(2).sub_(1).to(dtype)
    f = torch.full_like(u, float("nan"))
    f[1:n + 1, 1:n + 1] = torch.rand((n, n), generator=g, device="cuda:0", dtype=F64).to(dtype)
    return u, f


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 7, 8, 15, 16, 23, 24, 53, 54, 55, 107, 108, 109, 110,
                               215, 217, 512, 513, 649, 651, 799, 801, 949, 951, 1100, 1101, 2300])
def test_sweeps_equal_plain(n, dtype):
    print(f"windows n={n} {dtype}", flush=True)
    u0, f = grid(n, n, n + 2 + n % 5, dtype)
    for sweeps in (1, 2, 3, 4, 5, 6, 7, 9, 11, 13, 24):
        a, b = u0.clone(), u0.clone()
        rb.rbgs_sweep(a, f, sweeps)
        rb.rbgs_sweep(b, f, sweeps, kernel="plain")
        assert torch.equal(a, b), (n, sweeps)


@pytest.mark.parametrize("n,sweeps,dtype", [(3000, 1, F64), (4500, 24, F64), (4501, 8, F64),
                                            (4500, 1, F32), (10001, 7, F32)])
def test_short_calls_on_large_grids_equal_plain(n, sweeps, dtype):
    print(f"windows n={n} sweeps={sweeps} {dtype}", flush=True)
    u0, f = grid(n, n, n + 2, dtype)
    a, b = u0.clone(), u0
    rb.rbgs_sweep(a, f, sweeps)
    rb.rbgs_sweep(b, f, sweeps, kernel="plain")
    assert torch.equal(a, b)


@pytest.mark.parametrize("n", [1, 6, 31, 120, 255])
def test_sweeps_equal_oracle(oracle, n):
    h = W.spacing(n)
    u0 = W.random_ring(n, seed=n)
    f = W.uniform_rhs(n, seed=n + 1)
    ref = u0.copy()
    oracle.sweep(ref, f, h, 17)
    u = torch.from_numpy(u0.copy()).to("cuda:0")
    rb.rbgs_sweep(u, torch.from_numpy(f).to("cuda:0"), 17, h=h)
    assert np.array_equal(u.cpu().numpy(), ref)


@pytest.mark.parametrize("omega", [1.0, 1.7])
@pytest.mark.parametrize("n,check", [(40, 1), (40, 3), (129, 5), (129, 12), (700, 8), (1000, 25)])
def test_solves_equal_plain(n, check, omega):
    """Rounds of a solve (graph), a fixed count, and sweeps past the last whole
    round, Gauss-Seidel and SOR."""
    u0, f = grid(n, n, n + 2, F64)
    for max_sweeps, tol in ((4 * check + 2, 1e-30), (3 * check, 0.0)):
        a, b = u0.clone(), u0.clone()
        ia = rb.rbgs_solve(a, f, max_sweeps, tol, check_every=check, omega=omega)
        ib = rb.rbgs_solve(b, f, max_sweeps, tol, check_every=check, omega=omega, kernel="plain")
        assert ia == ib and torch.equal(a, b)


@pytest.mark.parametrize("precision", ["f32_ir", "bf16rhs_ir"])
def test_refinement_equals_plain(precision):
    n = 300
    u0, f = grid(n, 1, n + 2, F64)
    a, b = u0.clone(), u0.clone()
    ia = rb.rbgs_solve(a, f, 60, 1e-30, check_every=15, precision=precision)
    ib = rb.rbgs_solve(b, f, 60, 1e-30, check_every=15, precision=precision, kernel="plain")
    assert ia == ib and torch.equal(a, b)


@pytest.mark.parametrize("dtype", [F64, F32])
def test_split_layout_equals_plain(dtype):
    n = 333
    u, f = grid(n, 2, n + 2, dtype)
    ur, ub = rb.rbgs_pack(u)
    fr, fb = rb.rbgs_pack(f)
    for sweeps in (1, 5, 12):
        a, b = (ur.clone(), ub.clone()), (ur.clone(), ub.clone())
        rb.rbgs_sweep_split(n, *a, fr, fb, sweeps)
        rb.rbgs_sweep_split(n, *b, fr, fb, sweeps, kernel="plain")
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
