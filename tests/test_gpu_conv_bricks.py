"""The brick convolution against the per-voxel-tile kernel, bit for bit.

The two add an output's products in different orders, so the operands are whole numbers of at
most 3 (inputs) and 2 (weights): every partial sum is a whole number below 27 x 64 x 6 + 9 <
2^24, exact in binary32 in any order, and both kernels round the same value.  An input view
8 bytes off a 16-byte boundary takes the per-voxel-tile kernel.  The shapes take each brick:
8 x 8 x 8, 8 x 8 x 4 whole and cut at the upper x and y sides, 8 x 4 x 4 cut at x, 4 x 4 x 4;
the odd output stride takes its 2-byte stores, with weights 8 bytes off a 16-byte boundary."""
import pytest
import torch

from paper_1410_1921_amd import nn
from paper_1410_1921_amd.nn import View

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, nn.LBM_NN_RELU, nn.LBM_NN_FLIP])
@pytest.mark.parametrize("shape,cin,cout,ycs", [((48, 64, 64), 32, 16, 16), ((8, 40, 48), 16, 192, 200),
                                                ((36, 36, 36), 16, 64, 67), ((20, 28, 28), 48, 48, 96),
                                                ((12, 12, 12), 64, 128, 128), ((4, 4, 4), 16, 16, 17)])
def test_bricks_equal_tiles(shape, cin, cout, ycs, flags):
    nv = shape[0] * shape[1] * shape[2]
    gen = torch.Generator().manual_seed(nv + cin)
    x = torch.randint(-3, 4, (nv, cin), generator=gen).to(torch.bfloat16).cuda()
    xo = torch.zeros((nv, cin + 8), dtype=torch.bfloat16, device="cuda")
    xo[:, 4:4 + cin] = x
    off = 4 if ycs % 2 else 0
    w = torch.randint(-2, 3, (27 * cin * cout + off,), generator=gen).to(torch.bfloat16).cuda()[off:]
    bias = torch.randint(-9, 10, (cout,), generator=gen).float().cuda()
    ya = torch.full((nv, ycs), 7.0, dtype=torch.bfloat16, device="cuda")
    yb = ya.clone()
    nn.lbm_nn_conv3d(shape, View(x), cin, w, bias, View(ya, 0, cout), cout, flags)
    nn.lbm_nn_conv3d(shape, View(xo, 4, cin), cin, w, bias, View(yb, 0, cout), cout, flags)
    assert torch.equal(ya.view(torch.int16), yb.view(torch.int16))


@pytest.mark.parametrize("rows", [1, 40])
@pytest.mark.parametrize("shape,cin,cout", [((8, 16, 24), 16, 16), ((12, 12, 12), 64, 32), ((4, 4, 4), 16, 48),
                                            ((16, 28, 36), 32, 16), ((48, 48, 48), 16, 16)])
def test_weight_gradient_bricks_equal_tiles(shape, cin, cout, rows):
    """The same of the weight gradient: sums of at most 48^3 products of at most 6 and the
    accumulated start stay below 2^24.  A workspace of several times the size takes more
    chunks of bricks; 16 or more chunks take the sum with 16 threads an output."""
    nv = shape[0] * shape[1] * shape[2]
    gen = torch.Generator().manual_seed(nv + cout)
    x = torch.randint(-3, 4, (nv, cin), generator=gen).to(torch.bfloat16).cuda()
    xo = torch.zeros((nv, cin + 8), dtype=torch.bfloat16, device="cuda")
    xo[:, 4:4 + cin] = x
    g = torch.randint(-2, 3, (nv, cout), generator=gen).to(torch.bfloat16).cuda()
    size = nn.lbm_nn_wgrad_workspace(shape, cin, cout)
    out = []
    for view, ws in ((View(x), torch.empty(rows * size + 4, dtype=torch.uint8, device="cuda")[4:]),
                     (View(xo, 4, cin), torch.empty(size, dtype=torch.uint8, device="cuda"))):
        dw = torch.full((27 * cin * cout,), 5.0, device="cuda")
        db = torch.full((cout,), 5.0, device="cuda")
        nn.lbm_nn_conv3d_wgrad(shape, view, cin, View(g), cout, dw, db, ws, True)
        first = dw.clone()
        nn.lbm_nn_conv3d_wgrad(shape, view, cin, View(g), cout, dw, None, ws)
        out.append((first, dw, db))
    for a, b in zip(*out):
        assert torch.equal(a, b)
