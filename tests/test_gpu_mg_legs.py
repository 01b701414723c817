"""The fused legs of the multigrid cycle (automatic kernel) against the
oracle's cycle, bit for bit: sizes on both sides of a tile's 240 columns and of
its row strips, every split of the smoothing sweeps between the legs and the
half-sweeps before and after them, the switch to the one-workgroup coarse end
at 63, a Dirichlet ring, a wide row pitch, and a ring of f that must not be
read (NaN)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402


@pytest.mark.parametrize("n,nu1,nu2", [
    (65, 1, 1), (127, 2, 2), (131, 1, 2), (237, 2, 1), (239, 2, 2), (241, 2, 2), (243, 1, 1),
    (255, 3, 4), (479, 7, 1), (481, 1, 7), (511, 2, 3), (1025, 2, 2), (2049, 1, 1), (4001, 2, 2),
])
def test_legs_bitwise(oracle, n, nu1, nu2):
    print(f"mg legs n={n} nu=({nu1},{nu2})", flush=True)
    h, ld = W.spacing(n), n + 2 + n % 7
    u0 = W.random_ring(n, seed=n, ld=ld)
    u0[1:n + 1, 1:n + 1] = W.uniform_rhs(n, seed=n + 1)[1:n + 1, 1:n + 1]
    f = W.uniform_rhs(n, seed=n + 2, ld=ld)
    # levels of 63 and more are always present; an even coarsest level takes
    # few sweeps so that the oracle stays quick
    ref = u0.copy()
    _, _, rel = oracle.mg_solve(ref, f, h, nu1, nu2, 2, -1.0, coarse_sweeps=3)
    f[0, :], f[n + 1, :], f[:, 0], f[:, n + 1:] = np.nan, np.nan, np.nan, np.nan
    ut, ft = torch.from_numpy(u0).to("cuda:0"), torch.from_numpy(f).to("cuda:0")
    info = rb.rbgs_mg_solve(ut, ft, 2, -1.0, pre_sweeps=nu1, post_sweeps=nu2, coarse_sweeps=3, h=h)
    assert info["cycles"] == 2 and info["status"] == 0
    assert np.array_equal(ut.cpu().numpy(), ref)
    # a different order of n^2 additions of squares: at most n^2 roundings of 2^-53 each
    assert abs(info["rel_residual"] - rel) <= n * n * 2.0 ** -53 * rel
