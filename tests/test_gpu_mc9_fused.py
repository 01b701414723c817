"""The fused 9-point passes (automatic kernel) against the launch-per-colour
kernel and the oracle, bit for bit: sizes on both sides of a tile's columns
(58 or 60 pairs of columns) and strips, odd and even n, odd and even pass
counts and every depth, rounds of a solve, data that sends tiles to the exact
division (subnormal results), infinities and NaN, and a workspace that has no
second buffer."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402


def grid(n, seed, ld=None):
    u = W.random_ring(n, seed=seed, ld=ld)
    u[1:n + 1, 1:n + 1] = W.uniform_rhs(n, seed=seed + 1)[1:n + 1, 1:n + 1]
    return u, W.uniform_rhs(n, seed=seed + 2, ld=ld)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def same(a, b):
    """Equal bits, any NaN equal to any NaN."""
    return bool(torch.all((a.view(torch.int64) == b.view(torch.int64)) | (a.isnan() & b.isnan())))


@pytest.mark.parametrize("n,sweeps", [(1, 1), (1, 5), (2, 3), (3, 2), (7, 1), (118, 2), (119, 3),
                                      (120, 4), (121, 7), (239, 5), (240, 6), (241, 1), (1023, 4),
                                      (2999, 5), (3000, 4), (3001, 7), (3481, 6)])
def test_passes_bitwise(oracle, n, sweeps):
    print(f"mc9 passes n={n} sweeps={sweeps}", flush=True)
    h = W.spacing(n)
    u0, f = grid(n, n, ld=n + 2 + n % 3)
    ref = u0.copy()
    oracle.mc9_sweep(ref, f, h, sweeps)
    f[0, :], f[n + 1, :], f[:, 0], f[:, n + 1:] = np.nan, np.nan, np.nan, np.nan
    u = dev(u0)
    rb.rbgs_mc9_sweep(u, dev(f), sweeps, h=h)
    assert np.array_equal(u.cpu().numpy(), ref)


@pytest.mark.parametrize("case", ["subnormal", "front", "inf", "nan", "zero"])
@pytest.mark.parametrize("n", [63, 3001])
def test_unusual_values(n, case):
    print(f"mc9 unusual values {case} n={n}", flush=True)
    u0, f = grid(n, 5)
    if case == "subnormal":  # every result subnormal: ties of the division included
        rng = np.random.default_rng(1)
        u0 = rng.integers(-64, 65, size=u0.shape) * 5e-324
        f = np.zeros_like(f)
    elif case == "front":    # results from normal to subnormal to zero
        d = np.minimum(np.arange(n + 2)[:, None] + np.arange(n + 2)[None, :], 700)
        u0, f = 2.0 ** (-2.0 * d), np.zeros_like(f)
    elif case == "inf":
        u0[n // 2, n // 3], f[n // 4, n // 2] = np.inf, -np.inf
    elif case == "nan":
        u0[0, n // 2], f[n // 3, n // 3] = np.nan, np.nan
    else:                    # signed zeros
        u0 = np.where(np.indices(u0.shape).sum(0) % 3 == 0, -0.0, 0.0)
        f = np.where(np.indices(u0.shape).sum(0) % 5 == 0, -0.0, 0.0)
    a, b, ft = dev(u0), dev(u0), dev(f)
    rb.rbgs_mc9_sweep(a, ft, 7)
    rb.rbgs_mc9_sweep(b, ft, 7, kernel="plain")
    assert same(a, b)


@pytest.mark.parametrize("check", [1, 2, 3, 7])
def test_solve_rounds_equal_plain(check):
    n = 127
    u0, f = grid(n, 9)
    a, b, ft = dev(u0), dev(u0), dev(f)
    ia = rb.rbgs_mc9_solve(a, ft, 150, 1e-12, check_every=check)
    ib = rb.rbgs_mc9_solve(b, ft, 150, 1e-12, check_every=check, kernel="plain")
    assert ia == ib and same(a, b)


def test_workspace_without_second_buffer():
    n = 255
    u0, f = grid(n, 3)
    a, b, ft = dev(u0), dev(u0), dev(f)
    full = rb.rbgs_mc9_workspace_size(rb.make_grid(a))
    ld = (n + 2) // 2
    colour = ((n + 1) // 2 + 1) * ((ld + 1 + 31) // 32 * 32) * 8
    ws = torch.empty(full - 4 * ((colour + 255) // 256 * 256), dtype=torch.uint8, device="cuda:0")
    rb.rbgs_mc9_sweep(a, ft, 5, workspace=ws)
    rb.rbgs_mc9_sweep(b, ft, 5)
    assert same(a, b)
    with pytest.raises(rb.RbgsError):
        rb.rbgs_mc9_sweep(a, ft, 5, workspace=ws[:-256])
