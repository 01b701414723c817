"""Weight and bias gradients that come from one edge of the grid alone.

The target is the network's own output but for one row or column at the edge, so
that the loss gradient is zero everywhere else and an edge that a kernel drops or
shifts is a large part of the gradient, not the half percent that it is of a full
grid's sum: left out of one layer of the reference, it takes 0.18 to 1 of that
layer's bias gradient and 0.14 to 1 of its weights' (the first layer's, six layers
away, 0.08 at least) with it.  Stored values are BF16 on either side, which can move
each by 2^-8 of it, through 14 layers forward and 14 back: 28 * 2^-8 = 0.11 of the
gradient if all of them moved the same way.
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

TOL = 28 * 2.0 ** -8


def bf16(a):
    return torch.from_numpy(np.asarray(a, np.float64)).to(torch.bfloat16).to(torch.float64).numpy()


@pytest.mark.parametrize("factor,n", [(4, 191), (4, 255), (2, 127)])
def test_gradients_of_one_edge(factor, n):
    p = make_params(seed=6)
    net = rb.UNet(n, 1, factor=factor)
    net.set_params(flatten(p).astype(np.float32))
    f = batch_fields([5], n)
    ft = torch.from_numpy(f).to(DEV)
    out = torch.zeros_like(ft)
    net.forward(ft, out)
    _, _, cache, pr, rms = ref_forward(p, f[0], factor)
    amount = 1.0 + 0.5 * np.random.default_rng(2).random(n)
    for edge in ("first row", "last row", "first column", "last column"):
        say(f"unet edge gradients n={n} factor={factor} {edge}")
        d = np.zeros((n, n))
        at = 0 if "first" in edge else n - 1
        d[(at, slice(None)) if "row" in edge else (slice(None), at)] = amount
        target = out.clone()
        target[0, 1:-1, 1:-1] -= torch.from_numpy(d * rms).to(DEV)
        net.train_step(ft, target, 0.0, update=False)
        got = unflatten(net.get_grads().astype(np.float64), p)
        want = U.backward(pr, cache, 2.0 * d / (n * n), factor=factor, rnd=bf16)
        for k in want:
            rel = np.linalg.norm(got[k].ravel() - want[k].ravel()) / np.linalg.norm(want[k].ravel())
            assert rel < TOL, f"{edge}, {k}: relative L2 error {rel:.3e}"
