"""Calls on either side of the limits of the windows' rule, and the row pipeline
on large grids, bit for bit against the half-sweeps; the calls that were measured
slower there run the persistent kernel again."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402

F64, F32 = torch.float64, torch.float32


def grid(n, ld, dtype):
    g = torch.Generator(device="cuda:0").manual_seed(n)
    u = torch.rand((n + 2, ld), generator=g, device="cuda:0", dtype=dtype).mul_(2).sub_(1)
    f = torch.rand((n + 2, ld), generator=g, device="cuda:0", dtype=dtype).mul_(2).sub_(1)
    return u, f


@pytest.mark.parametrize("n,dtype,sweeps", [
    (5003, F64, (9, 20)), (8000, F64, (9, 16)), (8001, F64, (9, 30, 31)), (15501, F64, (9,)),
    (9200, F32, (8, 14)), (9201, F32, (8, 14, 15)), (10001, F32, (12, 14, 18, 20)),
])
def test_sweeps_equal_plain(n, dtype, sweeps):
    u, f = grid(n, n + 2 + n % 3, dtype)
    want, done = u.clone(), 0
    for k in sweeps:
        print(f"choice n={n} sweeps={k}", flush=True)
        rb.rbgs_sweep(want, f, k - done, kernel="plain")
        done = k
        got = u.clone()
        rb.rbgs_sweep(got, f, k)
        assert torch.equal(got, want), k


@pytest.mark.parametrize("n,dtype,sweeps", [
    (7500, F64, (2,)), (7501, F64, (2,)), (8100, F64, (9, 16)), (4300, F32, (14,)),
    (4301, F32, (14, 16)), (5501, F32, (2, 26, 28)), (7101, F32, (16,)),
])
def test_split_sweeps_equal_plain(n, dtype, sweeps):
    u, f = grid(n, n + 2, dtype)
    ur, ub = rb.rbgs_pack(u)
    fr, fb = rb.rbgs_pack(f)
    for k in sweeps:
        print(f"choice split n={n} sweeps={k}", flush=True)
        a, b = (ur.clone(), ub.clone()), (ur.clone(), ub.clone())
        rb.rbgs_sweep_split(n, *a, fr, fb, k)
        rb.rbgs_sweep_split(n, *b, fr, fb, k, kernel="plain")
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), k


@pytest.mark.parametrize("n,check,omega", [(1900, 2, 1.5), (1901, 2, 1.5), (8101, 9, 1.0)])
def test_solve_rounds_equal_plain(n, check, omega):
    u, f = grid(n, n + 2, F64)
    a, b = u.clone(), u
    ia = rb.rbgs_solve(a, f, 3 * check, 1e-30, check_every=check, omega=omega)
    ib = rb.rbgs_solve(b, f, 3 * check, 1e-30, check_every=check, omega=omega, kernel="plain")
    assert torch.equal(a, b) and ia == ib


@pytest.mark.parametrize("n,sweeps,persistent", [(10001, 14, True), (12501, 12, True),
                                                 (10001, 12, False), (9200, 14, False)])
def test_route(n, sweeps, persistent):
    u, f = grid(n, n + 2, F32)
    t = rb.rbgs_sweep(u, f, sweeps, timing=True)
    assert (t["persistent_launches"] > 0) == persistent
