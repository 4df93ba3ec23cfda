"""Network layers at sizes and channel strides beyond 32 bits: the network input where a thread per
group of channels would be more threads than a launch holds, and convolutions whose views put the
voxels of one brick further apart than 32-bit offsets reach."""
import pytest
import torch

from paper_1410_1921_amd import nn
from paper_1410_1921_amd.nn import View

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv,cs,off", [((1 << 22) + 5, 1024, 1),    # 1, 4, 8 channels a thread
                                       ((1 << 24) + 5, 1028, 4), ((1 << 25) + 5, 1024, 0)])
def test_network_input_beyond_a_launch(nv, cs, off):
    mask = (torch.arange(nv, device="cuda") % 3 == 0).to(torch.uint8)
    diam = torch.arange(nv, device="cuda", dtype=torch.float64) % 61
    x = torch.full((nv * cs + off,), 9.0, dtype=torch.bfloat16, device="cuda")[off:].view(nv, cs)
    print(nv, cs, off, flush=True)
    nn.lbm_nn_make_input(mask, diam, 4.0, View(x))
    assert torch.equal(x[:, 0], mask.to(torch.bfloat16))
    assert torch.equal(x[:, 1], (diam / 4.0).to(torch.float32).to(torch.bfloat16))
    for c in (2, 3, 7, 8, 511, cs - 1):
        assert not x[:, c].any(), c
    del x
    torch.cuda.empty_cache()
