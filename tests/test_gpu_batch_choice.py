"""FP64 batches of middle-sized and large grids on either way, windows (calls of few
sweeps, few grids) and persistent kernel (long calls of several large grids): which
one runs, and every grid bit for bit against the half-sweeps on it alone."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402


def batch(sizes, dtype):
    us, fs = [], []
    for k, n in enumerate(sizes):
        g = torch.Generator(device="cuda:0").manual_seed(n + k)
        for out in (us, fs):
            out.append(torch.rand((n + 2, n + 2 + k % 3), generator=g, device="cuda:0",
                                  dtype=dtype).mul_(2).sub_(1))
    return us, fs


def check(sizes, dtype, sweeps, **how):
    us, fs = batch(sizes, dtype)
    want, done = [u.clone() for u in us], 0
    for k in sweeps:
        print(f"batch choice {sizes} {dtype} x {k}", flush=True)
        for u, f in zip(want, fs):
            rb.rbgs_sweep(u, f, k - done, kernel="plain")
        done = k
        got = [u.clone() for u in us]
        t = rb.rbgs_sweep_batched(got, fs, k, timing=True, **how)
        for n, a, b in zip(sizes, got, want):
            assert torch.equal(a, b), (n, k)
    return t["sweep_launches"]


@pytest.mark.parametrize("sizes", [[1025, 2047, 60], [3001, 1535, 1536], [4095, 7, 2301], [4094]])
def test_windows_on_large_grids(sizes):
    assert check(sizes, torch.float64, (1, 2, 4, 5, 14, 20)) == 5  # passes of 20 sweeps


@pytest.mark.parametrize("sizes,sweeps", [([4095, 3500, 4000, 3900, 1], 100), ([2047] * 16, 45)])
def test_persistent_on_several_large_grids(sizes, sweeps):
    # passes of seven, and of what is left
    assert check(sizes, torch.float64, (sweeps,)) == 2


def test_fp32_windows():
    assert check([2600, 5001, 31], torch.float32, (6, 13)) == 3
