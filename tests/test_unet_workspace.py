"""The network's workspace: no larger than callers of the former size hold (the
layers' partial sums share a bounded part of it).  Host only."""
import pytest

from paper_2607_01735_amd import rbgs


@pytest.mark.parametrize("factor,n,batch,held", [
    (2, 63, 1, 24036096), (2, 63, 48, 250382592), (2, 255, 2, 135678720), (2, 255, 4, 251643136),
    (2, 511, 1, 240538368), (2, 511, 2, 459782912), (2, 1023, 1, 879219456),
    (4, 127, 8, 92289280), (4, 127, 24, 238240000), (4, 127, 128, 1186920448),
    (4, 127, 4096, 37382746624),
])
def test_former_workspaces_suffice(factor, n, batch, held):
    need = rbgs._lib.rbgs_unet_workspace_size(n, batch, factor)
    assert 0 < need <= held
