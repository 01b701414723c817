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
