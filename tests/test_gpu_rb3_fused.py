"""The fused 3D passes against the oracle and against the launch per
half-sweep (which a workspace without the second black array still runs), bit
for bit: sizes on both sides of a workgroup's 24 rows and 60 (62) columns, odd
and even n, odd and even pass counts, rounds of a solve, data that sends tiles
to the exact division (subnormal results), infinities, NaN and signed zeros,
a ring of f that must not be read, and a wide row pitch."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402


def grid(n, seed, ld=None):
    """u with a ring and f whose ring is NaN."""
    rng = np.random.default_rng(seed)
    shape = (n + 2, n + 2, ld or n + 2)
    u, f = rng.uniform(-1, 1, shape), np.full(shape, np.nan)
    f[1:n + 1, 1:n + 1, 1:n + 1] = rng.uniform(-1, 1, (n, n, n))
    return u, f


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def small_workspace(u, n):
    full = rb.rbgs_rb3_workspace_size(rb.make_grid3(u))
    pitch = ((n + 3) // 2 + 31) // 32 * 32
    return torch.empty(full - (n + 2) ** 2 * pitch * 8, dtype=torch.uint8, device="cuda:0")


def same(a, b):
    """Equal bits, any NaN equal to any NaN."""
    return bool(torch.all((a.view(torch.int64) == b.view(torch.int64)) | (a.isnan() & b.isnan())))


@pytest.mark.parametrize("n,sweeps", [(1, 1), (1, 4), (2, 3), (3, 2), (4, 5), (23, 2), (24, 3),
                                      (25, 4), (47, 1), (48, 6), (118, 3), (119, 2), (120, 4),
                                      (121, 5), (123, 1), (125, 1), (185, 2)])
def test_passes_bitwise(oracle, n, sweeps):
    print(f"rb3 passes n={n} sweeps={sweeps}", flush=True)
    h, ld = W.spacing(n), n + 2 + n % 3
    u0, f = grid(n, n, ld)
    f0 = np.where(np.isnan(f), 0.0, f)[:, :, :n + 2].copy()
    ref = u0[:, :, :n + 2].copy()
    oracle.rb3_sweep(ref, f0, h, sweeps)
    u = dev(u0)
    rb.rbgs_rb3_sweep(u, dev(f), sweeps, h=h)
    got = u.cpu().numpy()
    assert np.array_equal(got[:, :, :n + 2], ref)
    assert np.array_equal(got[:, :, n + 2:], u0[:, :, n + 2:])


@pytest.mark.parametrize("case", ["subnormal", "front", "inf", "nan", "zero"])
@pytest.mark.parametrize("n", [31, 130])
def test_unusual_values(n, case):
    print(f"rb3 unusual values {case} n={n}", flush=True)
    u0, f = grid(n, 5)
    inner = (slice(1, n + 1),) * 3
    if case == "subnormal":  # every result subnormal: ties of the division included
        u0 = np.random.default_rng(1).integers(-64, 65, size=u0.shape) * 5e-324
        f[inner] = 0.0
    elif case == "front":    # results from normal to subnormal to zero
        u0 = 2.0 ** (-4.0 * np.minimum(np.indices(u0.shape).sum(0), 300))
        f[inner] = 0.0
    elif case == "inf":
        u0[n // 2, n // 3, n // 4], f[n // 4, n // 2, n // 2] = np.inf, -np.inf
    elif case == "nan":
        u0[0, n // 2, n // 2], f[n // 3, n // 3, n // 2] = np.nan, np.nan
    else:                    # signed zeros
        u0 = np.where(np.indices(u0.shape).sum(0) % 3 == 0, -0.0, 0.0)
        f[inner] = np.where(np.indices((n, n, n)).sum(0) % 5 == 0, -0.0, 0.0)
    a, b, ft = dev(u0), dev(u0), dev(f)
    rb.rbgs_rb3_sweep(a, ft, 5)
    rb.rbgs_rb3_sweep(b, ft, 5, workspace=small_workspace(b, n))
    assert same(a, b)


@pytest.mark.parametrize("check", [1, 2, 3, 5])
def test_solve_rounds_equal_half_sweeps(check):
    n = 30
    u0, f = grid(n, 9)
    a, b, ft = dev(u0), dev(u0), dev(f)
    ia = rb.rbgs_rb3_solve(a, ft, 120, 1e-12, check_every=check)
    ib = rb.rbgs_rb3_solve(b, ft, 120, 1e-12, check_every=check, workspace=small_workspace(b, n))
    assert ia == ib and same(a, b)
