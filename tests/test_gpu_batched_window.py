"""Batches swept by register windows: sizes around a window's 64 columns and its
rows, every depth of pass, small and large batches, against the persistent
kernel, bit for bit, and a plan replayed with eager work in between."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402

DEV = torch.device("cuda:0")
SMALL = [1, 2, 3, 63, 64, 65, 100, 103, 104, 105, 127, 130, 255]
# enough points for the tall windows of each type (2e6 FP32, 8e5 FP64)
LARGE = [1023, 1, 700, 511, 64, 333, 900, 24, 2]


def batch(sizes, dtype):
    us = [W.random_ring(n, seed=50 + g, ld=n + 2 + g % 3).astype(dtype) for g, n in enumerate(sizes)]
    fs = [W.normal_rhs(n, seed=70 + g, ld=n + 2 + g % 3).astype(dtype) for g, n in enumerate(sizes)]
    return [[torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in x] for x in (us, fs)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("sizes", [SMALL, LARGE, [5]], ids=["small", "large", "one"])
def test_windows_equal_the_persistent_kernel(sizes, dtype):
    us, fs = batch(sizes, dtype)
    for nsweeps in (1, 2, 3, 4, 5, 6, 7, 11, 13, 25):
        print(f"windows {np.dtype(dtype)} {len(sizes)} grids {nsweeps} sweeps", flush=True)
        a, b = [u.clone() for u in us], [u.clone() for u in us]
        rb.rbgs_sweep_batched(a, fs, nsweeps)
        rb.rbgs_sweep_batched(b, fs, nsweeps, kernel="blocked")
        for g, n in enumerate(sizes):
            assert torch.equal(a[g], b[g]), f"{nsweeps} sweeps, grid {g} (n={n})"


@pytest.mark.parametrize("nsweeps", [6, 17])
def test_plan_replays(nsweeps):
    print(f"window plan {nsweeps} sweeps", flush=True)
    us, fs = batch(SMALL, np.float32)
    a, b = [u.clone() for u in us], [u.clone() for u in us]
    plan = rb.BatchPlan(a, fs, nsweeps)
    for r in range(3):
        for x in a + b:  # the program's own work between replays
            x[1:-1, 1:-1].mul_(0.5)
        plan.launch()
        plan.check()
        rb.rbgs_sweep_batched(b, fs, nsweeps, kernel="blocked")
        torch.cuda.synchronize()
        for g, n in enumerate(SMALL):
            assert torch.equal(a[g], b[g]), f"replay {r}, grid {g} (n={n})"
    plan.close()


@pytest.mark.parametrize("precision,omega", [("f64", 1.0), ("f32_ir", 1.0), ("f64", 1.5)])
def test_batched_solves_equal_the_persistent_kernel(precision, omega):
    """Rounds of 25 sweeps (an odd number of passes), grids that leave early,
    and a last round cut short by the sweep budget."""
    print(f"batched solve {precision} omega={omega}", flush=True)
    sizes = [3, 15, 63, 64, 31, 7]
    us, fs = batch(sizes, np.float64)
    a, b = [u.clone() for u in us], [u.clone() for u in us]
    kw = dict(precision=precision, omega=omega)
    ia = rb.rbgs_solve_batched(a, fs, 310, 1e-6, 25, **kw)
    ib = rb.rbgs_solve_batched(b, fs, 310, 1e-6, 25, kernel="blocked", **kw)
    for g, n in enumerate(sizes):
        assert torch.equal(a[g], b[g]), f"grid {g} (n={n})"
        assert ia[g]["sweeps"] == ib[g]["sweeps"]
        assert ia[g]["rel_residual"] == ib[g]["rel_residual"]
