"""Parameters and gradients to the host around the sizes where the copy
changes: below a ring, a ring's worth and past it, pageable and pinned
destinations, two threads at once."""
import ctypes as C
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("base,levels", [(16, 1), (64, 2), (48, 3), (64, 3)])   # 0.1, 4.3, 7.7, 14 MB
def test_params_come_back(base, levels):
    from paper_1812_06632_amd import soc
    ctx = soc.Context(0)
    net = soc.UNet(ctx, 2, 2, base, levels, 1, (8, 8, 8))
    p = np.random.default_rng(base).standard_normal(net.param_count).astype(np.float32)
    net.set_params(p)
    for _ in range(3):
        assert np.array_equal(net.get_params(), p)
    pinned = torch.empty(net.param_count, dtype=torch.float32, pin_memory=True)
    ctx.check(soc._lib.soc_unet_get_params(ctx.h, net.h, C.c_void_p(pinned.data_ptr())))
    assert np.array_equal(pinned.numpy(), p)
    got = [None, None]

    def get(i):
        got[i] = net.get_params()
    threads = [threading.Thread(target=get, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(np.array_equal(g, p) for g in got)
    ctx.close()
