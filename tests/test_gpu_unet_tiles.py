"""The U-Net's 3^3 convolutions in every form of their dispatch (planes per
wave, channels per chunk, column tiles), on grids that end inside a brick,
per element against the FP64 layers on the device's own stored tensors."""
import numpy as np
import pytest

from tests.test_gpu_unet import _case, flat, soc  # noqa: F401
from tests.unet_parity import check_backward_layers, check_forward_layers, print_rows

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("base,n,shape", [
    (16, 1, (1, 1, 1)),         # one cell
    (16, 1, (3, 5, 9)),         # one plane per wave, 32 channels per chunk, one column tile
    (48, 1, (9, 10, 11)),       # a last chunk of 16 channels, two column tiles
    (16, 1, (40, 47, 37)),      # two planes per wave
    (64, 1, (31, 30, 26)),      # two planes, two column tiles
    (64, 1, (18, 26, 27)),      # one plane, two column tiles
    (80, 1, (20, 26, 27)),      # the same, a last chunk of 16 channels
    (64, 1, (5, 9, 10)),        # 64 columns, one column tile
    (16, 1, (2, 128, 121)),     # 16 channels per chunk, one plane
    (16, 1, (66, 61, 34)),      # four planes, one column tile
    (64, 1, (50, 51, 33)),      # four planes, two column tiles
])
def test_layers_match_oracle(soc, base, n, shape):  # noqa: F811
    P, x, dy = _case(1, base, n, shape, seed=base)
    ctx = soc.Context(0)
    net = soc.UNet(ctx, 2, 2, base, 1, n, shape)
    net.set_params(flat(P).astype(np.float32))
    y = net.forward(torch.from_numpy(x.astype(np.float32)).cuda()).cpu().numpy().astype(np.float64)
    rep = check_forward_layers(net, P, n, shape, 2, 2, base, 1, y)
    rep += check_backward_layers(net, P, torch.from_numpy(dy.astype(np.float32)).cuda(), n, shape, 2, 2, base, 1)
    print_rows(rep)
    ctx.close()


@pytest.mark.parametrize("levels,n,shape", [(2, 2, (6, 10, 14)), (3, 1, (12, 20, 28))])
def test_down_and_up_on_odd_grids(soc, levels, n, shape):  # noqa: F811
    P, x, dy = _case(levels, 16, n, shape, seed=levels)
    ctx = soc.Context(0)
    net = soc.UNet(ctx, 2, 2, 16, levels, n, shape)
    net.set_params(flat(P).astype(np.float32))
    y = net.forward(torch.from_numpy(x.astype(np.float32)).cuda()).cpu().numpy().astype(np.float64)
    rep = check_forward_layers(net, P, n, shape, 2, 2, 16, levels, y)
    rep += check_backward_layers(net, P, torch.from_numpy(dy.astype(np.float32)).cuda(), n, shape, 2, 2, 16, levels)
    print_rows(rep)
    ctx.close()


@pytest.mark.parametrize("base,shape", [
    (16, (66, 62, 66)),         # up and down: one column tile, two phases per wave
    (64, (64, 62, 68)),         # two column tiles
    (48, (10, 6, 14)),          # an odd number of 16 channels, one phase per wave
])
def test_between_levels(soc, base, shape):  # noqa: F811
    P, x, dy = _case(2, base, 1, shape, seed=base)
    ctx = soc.Context(0)
    net = soc.UNet(ctx, 2, 2, base, 2, 1, shape)
    net.set_params(flat(P).astype(np.float32))
    y = net.forward(torch.from_numpy(x.astype(np.float32)).cuda()).cpu().numpy().astype(np.float64)
    rep = check_forward_layers(net, P, 1, shape, 2, 2, base, 2, y)
    rep += check_backward_layers(net, P, torch.from_numpy(dy.astype(np.float32)).cuda(), 1, shape, 2, 2, base, 2)
    print_rows(rep)
    ctx.close()


@pytest.mark.parametrize("cin,cout", [(1, 1), (7, 9), (17, 16)])   # channels padded to 16 and 32, 8 at a time
def test_odd_channels(soc, cin, cout):  # noqa: F811
    n, shape = 2, (4, 6, 10)
    P, x, dy = _case(2, 16, n, shape, cin, cout, seed=cin)
    ctx = soc.Context(0)
    net = soc.UNet(ctx, cin, cout, 16, 2, n, shape)
    net.set_params(flat(P).astype(np.float32))
    y = net.forward(torch.from_numpy(x.astype(np.float32)).cuda()).cpu().numpy().astype(np.float64)
    rep = check_forward_layers(net, P, n, shape, cin, cout, 16, 2, y)
    rep += check_backward_layers(net, P, torch.from_numpy(dy.astype(np.float32)).cuda(), n, shape, cin, cout, 16, 2)
    print_rows(rep)
    ctx.close()


@pytest.mark.parametrize("cout", [31, 32, 33, 48, 64, 65, 100])   # column tiles of 32, the last one full, partial or padding
@pytest.mark.parametrize("shape", [(3, 5, 9), (2, 128, 121)])      # one column tile per workgroup, and two
def test_wide_outputs(soc, cout, shape):  # noqa: F811
    P, x, dy = _case(1, 16, 1, shape, 2, cout, seed=cout)
    ctx = soc.Context(0)
    net = soc.UNet(ctx, 2, cout, 16, 1, 1, shape)
    net.set_params(flat(P).astype(np.float32))
    y = net.forward(torch.from_numpy(x.astype(np.float32)).cuda()).cpu().numpy().astype(np.float64)
    rep = check_forward_layers(net, P, 1, shape, 2, cout, 16, 1, y)
    rep += check_backward_layers(net, P, torch.from_numpy(dy.astype(np.float32)).cuda(), 1, shape, 2, cout, 16, 1)
    print_rows(rep)
    ctx.close()


@pytest.mark.parametrize("base,levels,shape,nmax", [
    (48, 2, (16, 16, 16), 3),   # more weight-gradient chunks for two samples than for three
    (16, 1, (24, 24, 24), 5),   # for three and four than for five
])
def test_smaller_batches_than_the_network_was_made_for(soc, base, levels, shape, nmax):  # noqa: F811
    """Every batch up to nmax gives the gradients of a network made for it."""
    P, x, dy = _case(levels, base, nmax, shape, seed=nmax)
    xt, dyt = (torch.from_numpy(v.astype(np.float32)).cuda() for v in (x, dy))
    ctx = soc.Context(0)
    large = soc.UNet(ctx, 2, 2, base, levels, nmax, shape)
    large.set_params(flat(P).astype(np.float32))
    for n in range(1, nmax + 1):
        own = soc.UNet(ctx, 2, 2, base, levels, n, shape)
        own.set_params(flat(P).astype(np.float32))
        got = []
        for net in (large, own):
            y = net.forward(xt[:n].contiguous())
            net.backward(dyt[:n].contiguous())
            got.append((y.cpu().numpy(), net.get_grads()))
        assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
        own.close()
    ctx.close()
