"""FP64 sweeps by row-walking tiles, a launch a pass: sizes around the limits
of the rule, every depth of pass, odd and even numbers of passes, SOR and
captured rounds, against one launch per half-sweep, bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402

DEV = torch.device("cuda:0")


def grid(n, ld):
    u = torch.from_numpy(np.ascontiguousarray(W.random_ring(n, seed=n, ld=ld))).to(DEV)
    f = torch.from_numpy(np.ascontiguousarray(W.normal_rhs(n, seed=n + 1, ld=ld))).to(DEV)
    return u, f


@pytest.mark.parametrize("n,ld", [(1600, 1602), (1601, 1605), (2047, 2049), (3501, 3503),
                                  (4502, 4504)])
def test_sweeps_equal_plain(n, ld):
    u, f = grid(n, ld)
    want, done = u.clone(), 0
    for nsweeps in (9, 10, 11, 13, 15, 21, 28):  # depths 2 .. 7 over the sizes
        print(f"pipeline n={n} sweeps={nsweeps}", flush=True)
        rb.rbgs_sweep(want, f, nsweeps - done, kernel="plain")
        done = nsweeps
        got = u.clone()
        rb.rbgs_sweep(got, f, nsweeps)
        assert torch.equal(got, want), f"{nsweeps} sweeps"


@pytest.mark.parametrize("check", [11, 15, 20])
@pytest.mark.parametrize("omega", [1.0, 1.7])
def test_solve_rounds_equal_plain(check, omega):
    print(f"pipeline solve check={check} omega={omega}", flush=True)
    u, f = grid(1803, 1805)
    a, b = u.clone(), u.clone()
    ia = rb.rbgs_solve(a, f, 3 * check, 1e-30, check_every=check, omega=omega)
    ib = rb.rbgs_solve(b, f, 3 * check, 1e-30, check_every=check, omega=omega, kernel="plain")
    assert torch.equal(a, b)
    assert ia["sweeps"] == ib["sweeps"] and ia["rel_residual"] == ib["rel_residual"]
