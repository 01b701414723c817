"""3D kernel choice: PLAIN is a launch per half-sweep and never touches the fused
passes' second black array, AUTO (the default) takes the passes; the same bits."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402

MARK = 0x5a


def problem(n, seed=0):
    rng = np.random.default_rng(seed)
    u = rng.uniform(-1, 1, (n + 2,) * 3)
    f = rng.uniform(-1, 1, (n + 2,) * 3)
    return u, f


def workspace(u, n):
    """A workspace filled with a mark, and its second black array (at the end)."""
    pitch = ((n + 3) // 2 + 31) // 32 * 32
    size = rb.rbgs_rb3_workspace_size(rb.make_grid3(u))
    ws = torch.full((size,), MARK, dtype=torch.uint8, device="cuda:0")
    return ws, ws[size - (n + 2) ** 2 * pitch * 8:]


@pytest.mark.parametrize("kernel,fused", [("plain", False), ("resident", False), ("auto", True),
                                          (None, True)])
@pytest.mark.parametrize("call", ["sweep", "fixed", "rounds"])
def test_kernel_is_the_one_asked_for(oracle, kernel, fused, call):
    print(f"rb3 kernel={kernel} {call}", flush=True)
    n, sweeps = 20, 12
    h = W.spacing(n)
    u0, f = problem(n)
    ref = oracle.rb3_sweep(u0.copy(), f, h, sweeps)
    u, ft = torch.from_numpy(u0.copy()).to("cuda:0"), torch.from_numpy(f).to("cuda:0")
    ws, second = workspace(u, n)
    how = {} if kernel is None else {"kernel": kernel}
    if call == "sweep":
        rb.rbgs_rb3_sweep(u, ft, sweeps, h=h, workspace=ws, **how)
    else:
        tol = -1.0 if call == "fixed" else 1e-30
        rb.rbgs_rb3_solve(u, ft, sweeps, tol, check_every=4, h=h, workspace=ws, **how)
    assert np.array_equal(u.cpu().numpy(), ref)
    assert bool((second != MARK).any()) == fused


@pytest.mark.parametrize("n,sweeps,fused", [(1, 20, True), (2, 3, False), (7, 2, True), (7, 3, False),
                                            (7, 20, False), (8, 20, True)])
def test_tiny_grids_take_half_sweeps(oracle, n, sweeps, fused):
    """A pass's steps take longer than the launches they save there."""
    print(f"rb3 tiny n={n} x {sweeps}", flush=True)
    h = W.spacing(n)
    u0, f = problem(n)
    ref = oracle.rb3_sweep(u0.copy(), f, h, sweeps)
    ft = torch.from_numpy(f).to("cuda:0")
    u = torch.from_numpy(u0.copy()).to("cuda:0")
    ws, second = workspace(u, n)
    rb.rbgs_rb3_sweep(u, ft, sweeps, h=h, workspace=ws)
    assert np.array_equal(u.cpu().numpy(), ref)
    # black's ring goes there either way, the interior point (1, 1, 1) only with passes
    point = second.view(torch.int64).reshape(n + 2, n + 2, -1)[1, 1, 0].item()
    assert (point != 0x5a5a5a5a5a5a5a5a) == fused
    u = torch.from_numpy(u0.copy()).to("cuda:0")
    rb.rbgs_rb3_solve(u, ft, sweeps, -1.0, check_every=sweeps, h=h)
    assert np.array_equal(u.cpu().numpy(), ref)


@pytest.mark.parametrize("n,fused", [(699, True), (700, False)])
def test_one_sweep_of_a_large_grid(n, fused):
    print(f"rb3 one sweep n={n}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    u = torch.rand((n + 2,) * 3, generator=g, device="cuda:0", dtype=torch.float64)
    f = torch.zeros_like(u)
    want = u.clone()
    rb.rbgs_rb3_sweep(want, f, 1, kernel="plain")
    ws, second = workspace(u, n)
    rb.rbgs_rb3_sweep(u, f, 1, workspace=ws)
    assert torch.equal(u, want)
    point = second.view(torch.int64).reshape(n + 2, n + 2, -1)[1, 1, 0].item()
    assert (point != 0x5a5a5a5a5a5a5a5a) == fused
