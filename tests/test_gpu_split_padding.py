"""Split arrays belong to the caller, entries past column n + 1 included: an odd
number of persistent passes, whose result is copied back from the workspace, leaves
those entries alone."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402


@pytest.mark.parametrize("dtype,code", [(torch.float64, 0), (torch.float32, 1)])
@pytest.mark.parametrize("n", [1, 8, 61, 62, 63, 253, 254, 333])
def test_padding_is_left_alone(n, dtype, code):
    print(f"split padding n={n} {dtype}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    u = torch.rand((n + 2, n + 2), generator=g, device="cuda:0", dtype=dtype)
    f = torch.rand((n + 2, n + 2), generator=g, device="cuda:0", dtype=dtype)
    ur, ub = rb.rbgs_pack(u)
    fr, fb = rb.rbgs_pack(f)
    width = (n + 3) // 2
    for c in (ur, ub):
        c[:, width:] = 7.0
    want = (ur.clone(), ub.clone())
    rb.rbgs_sweep_split(n, *want, fr, fb, 5, kernel="plain")
    ws = torch.full((rb.rbgs_workspace_size(rb.make_grid(u), code),), 255, dtype=torch.uint8,
                    device="cuda:0")
    rb.rbgs_sweep_split(n, ur, ub, fr, fb, 5, kernel="blocked", fuse=2, workspace=ws)
    assert torch.equal(ur, want[0]) and torch.equal(ub, want[1])
