"""Gradients whose partial sums do not all fit their part of the workspace are added
in several launches: the same bits as in one.  A network created for one batch has
little room, one created for many has enough for a small batch's."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2607_01735_amd as rb  # noqa: E402


@pytest.mark.parametrize("factor,n,batch,room", [(2, 63, 1, 24), (2, 63, 3, 64), (2, 127, 2, 16),
                                                 (4, 127, 8, 48), (4, 191, 1, 8)])
def test_same_gradients(factor, n, batch, room):
    print(f"unet partials F={factor} n={n} batch={batch}", flush=True)
    f = torch.stack([torch.from_numpy(W.uniform_rhs(n, seed=k)) for k in range(batch)]).to("cuda:0")
    t = torch.stack([torch.from_numpy(W.uniform_rhs(n, seed=90 + k)) for k in range(batch)]).to("cuda:0")
    count = rb.UNet(n, 1, factor=factor).count
    params = (np.random.default_rng(n).standard_normal(count) * 0.05).astype(np.float32)
    grads = []
    for capacity in (batch, room):
        net = rb.UNet(n, capacity, factor=factor)
        net.set_params(params)
        for _ in range(2):
            net.train_step(f, t, 0.0)
        grads.append(net.get_grads())
    assert np.any(grads[0]) and np.array_equal(grads[0], grads[1])
