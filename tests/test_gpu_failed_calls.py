"""Calls after one that failed: the runtime error that a refused allocation
leaves does not reach the next, nor does what a call had done before it
failed."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _problem():
    from paper_1812_06632_amd import soc, workloads as W

    P = W.sphere_problem(n=8, n_packages=1000)
    ctx = soc.Context(0)
    grid = soc.grid_from_workload(ctx, P.grid)
    f = (float(P.nu[0]), float(P.w[0]), float(P.sigma_abs[0]), float(P.sigma_sca[0]), float(P.g[0]))
    return soc, P, ctx, grid, f


def test_scratch_that_cannot_be_had():
    """80 frequencies of 2^31 - 1 weighted packages need 687 GB of package
    lists; the call after the refusal runs."""
    soc, P, ctx, grid, f = _problem()
    A = torch.zeros(P.grid.ncells, dtype=torch.float64, device="cuda")
    T = torch.full((P.grid.ncells,), 20.0, dtype=torch.float32, device="cuda")
    src = dict(T=T, n_dust=2**31 - 1)
    with pytest.raises(soc.SocError) as e:
        soc.simulate_frequencies(ctx, grid, [f] * 80, A, [src] * 80, range(80), seed=1, iteration=1)
    assert e.value.status == soc.ENOMEM
    st = soc.simulate_frequency(ctx, grid, f, A, I_bg=float(P.I_bg[0]), n_bg=1000, seed=3, stats=True)
    assert st["packages"] == 1000


def test_network_that_cannot_be_had():
    """2^26 cells of 4096 channels need 550 GB for one tensor."""
    soc, P, ctx, grid, f = _problem()
    with pytest.raises(soc.SocError) as e:
        soc.UNet(ctx, 1, 1, 4096, 1, 256, (64, 64, 64))
    assert e.value.status == soc.ENOMEM
    net = soc.UNet(ctx, 1, 1, 16, 1, 1, (4, 4, 4))
    assert torch.isfinite(net.forward(torch.ones(1, 4, 4, 4, 1, device="cuda"))).all()


def _leave_an_error():
    """A pending error of the HIP runtime, as a program's own refused allocation leaves it."""
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    p = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 62)) != 0


def test_temperature_statistics_after_a_failed_call():
    soc, P, ctx, grid, f = _problem()
    table = soc.temp_table_build(ctx, P.emit_nu, P.emit_w, P.emit_sigma_abs, P.T_floor, P.T_max, 1024)
    T = torch.linspace(5, 50, P.grid.ncells, device="cuda")
    want = soc.temperature_stats(ctx, grid, table, T)
    _leave_an_error()
    try:
        assert soc.temperature_stats(ctx, grid, table, T) == want
    except soc.SocError as e:
        assert e.status == soc.EHIP
    assert soc.temperature_stats(ctx, grid, table, T) == want
