"""The U-Net's convolution kernels at the sizes where their tiles end.

Levels of 191 / 47 / 11 / 2 and 255 / 63 / 15 / 3 points (coarsening 4) and
127 / 63 / 31 / 15 (coarsening 2) leave remainders of every kind in the
16-pixel groups, the strips and the row bands; the batch decides how many
outputs a wave takes.  An output's sum has one order, whatever the batch, so
the samples of a batch are the samples alone, bit for bit; against the FP64
reference with BF16 storage what is left is FP32 summation, which can move a
stored value across a rounding boundary: at most 2^-8 of it, in each of 14
layers, 1.5e-2 in all if every value of every layer moved.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402
from oracle import unet_ref as U  # noqa: E402
from tests.test_gpu_unet import (DEV, batch_fields, flatten, make_params, ref_forward,  # noqa: E402
                                 say, unflatten)

TOL = 14 ** 0.5 * 2.0 ** -8


@pytest.mark.parametrize("factor,n,batch", [(4, 191, 3), (4, 255, 8), (2, 127, 5)])
def test_batch_is_its_samples_and_matches_reference(factor, n, batch):
    say(f"unet conv n={n} factor={factor} batch={batch}")
    p = make_params(seed=3)
    net = rb.UNet(n, batch, factor=factor)
    net.set_params(flatten(p).astype(np.float32))
    f = batch_fields(range(batch), n)
    ft = torch.from_numpy(f).to(DEV)
    u0 = torch.zeros_like(ft)
    net.forward(ft, u0)
    one = torch.zeros_like(ft[:1])
    for b in range(batch):
        net.forward(ft[b:b + 1].contiguous(), one)
        assert torch.equal(one[0], u0[b]), f"sample {b}"
    ref = ref_forward(p, f[0], factor)[0]
    err = np.linalg.norm(u0[0, 1:-1, 1:-1].cpu().numpy() - ref) / np.linalg.norm(ref)
    say(f"relative L2 error {err:.3e}")
    assert err < TOL


@pytest.mark.parametrize("factor,n", [(4, 191), (2, 127)])
def test_gradients_at_tile_edges(factor, n):
    say(f"unet gradients n={n} factor={factor}")
    p = make_params(seed=4)
    net = rb.UNet(n, 1, factor=factor)
    net.set_params(flatten(p).astype(np.float32))
    f = batch_fields([3], n)
    target = np.zeros_like(f)
    target[:, 1:-1, 1:-1] = np.random.default_rng(8).standard_normal((1, n, n)) * 0.01
    net.train_step(torch.from_numpy(f).to(DEV), torch.from_numpy(target).to(DEV), 0.0, update=False)
    got = unflatten(net.get_grads().astype(np.float64), p)
    _, y, cache, pr, rms = ref_forward(p, f[0], factor)
    _, dy = U.mse_loss(y, target[0, 1:-1, 1:-1] / rms)
    want = U.backward(pr, cache, dy, factor=factor, rnd=lambda a: torch.from_numpy(
        np.asarray(a, np.float64)).to(torch.bfloat16).to(torch.float64).numpy())
    for k in want:
        rel = np.linalg.norm(got[k].ravel() - want[k].ravel()) / np.linalg.norm(want[k].ravel())
        assert rel < TOL, f"{k}: relative L2 error {rel:.3e}"


def test_gradient_of_a_batch_is_the_mean_of_its_samples():
    """Eight samples of 255^2 walk down bands of 16 rows, one alone bands of
    four.  The loss is a mean over 8 = 2^3 samples, so the stored gradients of
    a sample are the same numbers times 1/8; the weight gradients differ by
    FP32 sums of about 100 roundings, 6e-6 of their terms' magnitudes, which
    are taken to be at most 16 times the result's."""
    say("unet batch gradient")
    n, batch = 255, 8
    p = make_params(seed=5)
    net = rb.UNet(n, batch, factor=4)
    net.set_params(flatten(p).astype(np.float32))
    f = torch.from_numpy(batch_fields(range(batch), n)).to(DEV)
    g = torch.Generator().manual_seed(1)
    target = torch.zeros_like(f)
    target[:, 1:-1, 1:-1] = (torch.randn(batch, n, n, generator=g, dtype=torch.float64) * 0.01).to(DEV)
    net.train_step(f, target, 0.0, update=False)
    got = unflatten(net.get_grads().astype(np.float64), p)
    total = 0.0
    for b in range(batch):
        net.train_step(f[b:b + 1].contiguous(), target[b:b + 1].contiguous(), 0.0, update=False)
        total = total + net.get_grads().astype(np.float64) / batch
    want = unflatten(total, p)
    for k in want:
        rel = np.linalg.norm(got[k].ravel() - want[k].ravel()) / np.linalg.norm(want[k].ravel())
        assert rel < 1e-4, f"{k}: relative L2 error {rel:.3e}"
