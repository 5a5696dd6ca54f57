"""Temperature solve and its statistics at the sizes where the passes
change: one cell, partial workgroups, both sides of the LDS-staged form,
and fields at and beyond the table's ends."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

T_FLOOR, T_MAX = 2.0, 3000.0


def _setup(nx, ny, nz, nT=4096):
    from paper_1812_06632_amd import soc, workloads as W

    ctx = soc.Context(0)
    rng = np.random.default_rng(nx * 131 + ny)
    rho = rng.uniform(0.5, 2.0, (nz, ny, nx))
    if rho.size > 1:
        rho[rng.random(rho.shape) < 0.05] = 0.0
    g = W.regular_grid(rho.astype(np.float32), 1e16)
    grid = soc.grid_from_workload(ctx, g)
    nu, w = W.frequency_grid(24)
    sabs, _, _ = W.dust_model(nu)
    table = soc.temp_table_build(ctx, nu, w, sabs, T_FLOOR, T_MAX, nT)
    return soc, W, ctx, g, grid, table, (nu, w, sabs)


def _gamma(W, T, nu, w, sabs):
    return 4 * math.pi * sum(b * c * W._bb(a, T) for a, b, c in zip(nu, w, sabs))


def _hot5(T):
    k = math.ceil(0.05 * T.size)
    return float(np.sort(T.astype(np.float64))[::-1][:k].mean())


# 512-lane workgroups; the LDS-staged form from 2048 cells per workgroup of at most 512 workgroups
@pytest.mark.parametrize("shape", [(1, 1, 1), (7, 3, 3), (8, 8, 8), (23, 27, 13), (101, 101, 101), (103, 102, 101)])
@pytest.mark.parametrize("nT", [16, 4096])
def test_solve_and_statistics(shape, nT):
    soc, W, ctx, g, grid, table, model = _setup(*shape, nT=nT)
    rng = np.random.default_rng(3)
    n = g.ncells
    dens = g.density().astype(np.float64)
    # on the table's own temperatures interpolation adds nothing: the solve returns them
    lnT = np.linspace(math.log(T_FLOOR), math.log(T_MAX), nT)
    want = np.exp(lnT[rng.integers(1, nT - 1, n)])
    A = np.where(dens > 0, _gamma(W, want, *model) * dens * 1e16 ** 3, 0.0)
    cold, hot = rng.random(n) < 0.02, rng.random(n) < 0.02
    A[cold] = 0.0
    A[hot & ~cold] *= 1e30
    want = np.where(cold, T_FLOOR, np.where(hot, T_MAX, want))
    want[dens == 0] = 0.0
    old = np.where(rng.random(n) < 0.1, 0.0, rng.uniform(5, 50, n)).astype(np.float32)
    T = torch.empty(n, dtype=torch.float32, device="cuda")
    At, oldt = torch.from_numpy(A).cuda(), torch.from_numpy(old).cuda()
    for _ in range(2):   # the second call finds the histograms as the first one left them
        st = soc.update_temperature(ctx, grid, table, At, T, oldt, stats=True)
    got = T.cpu().numpy()
    # FP64 tables of the same sum, then one rounding to FP32
    np.testing.assert_allclose(got, want, rtol=1e-6)
    leaf = dens > 0
    v = got[leaf].astype(np.float64)
    assert st["mean_T"] == pytest.approx(v.mean(), rel=1e-12)
    # a fine bin of the threshold holds 4 neighbouring floats at most
    assert st["hot5_mean_T"] == pytest.approx(_hot5(got[leaf]), rel=5e-7)
    assert st["clamped"] == int((leaf & (cold | hot)).sum())
    both = leaf & (old > 0)
    if both.any():
        rel = np.abs(got[both].astype(np.float64) - old[both]) / old[both]
        assert st["mean_rel_change"] == pytest.approx(rel.mean(), rel=1e-12)
    else:
        assert math.isnan(st["mean_rel_change"])
    # without statistics the same temperatures
    T2 = torch.empty_like(T)
    soc.update_temperature(ctx, grid, table, At, T2)
    assert torch.equal(T, T2)


@pytest.mark.parametrize("field", ["zeros", "equal", "beyond", "ties"])
def test_statistics_of_given_fields(field):
    soc, W, ctx, g, grid, table, _ = _setup(23, 27, 13)
    rng = np.random.default_rng(5)
    n = g.ncells
    T = {"zeros": np.zeros(n), "equal": np.full(n, 17.25),
         "beyond": np.where(rng.random(n) < 0.2, 4000.0, rng.uniform(0.5, 30.0, n)),
         "ties": rng.integers(10, 14, n).astype(np.float64)}[field].astype(np.float32)
    leaf = g.density() > 0
    st = soc.temperature_stats(ctx, grid, table, torch.from_numpy(T).cuda())
    assert st["mean_T"] == pytest.approx(T[leaf].astype(np.float64).mean(), rel=1e-12)
    assert st["hot5_mean_T"] == pytest.approx(_hot5(T[leaf]), rel=5e-7)


@pytest.mark.parametrize("share", [0.02, 0.2, 1.0])   # above the threshold's bin, in it, everywhere
def test_statistics_of_infinite_temperatures(share):
    soc, W, ctx, g, grid, table, _ = _setup(23, 27, 13)
    rng = np.random.default_rng(9)
    T = rng.uniform(5.0, 30.0, g.ncells).astype(np.float32)
    T[rng.random(g.ncells) < share] = np.inf
    st = soc.temperature_stats(ctx, grid, table, torch.from_numpy(T).cuda())
    assert st["mean_T"] == np.inf and st["hot5_mean_T"] == np.inf
    T[~np.isfinite(T)] = 20.0   # nothing of it is left in the next call
    st = soc.temperature_stats(ctx, grid, table, torch.from_numpy(T).cuda())
    assert st["hot5_mean_T"] == pytest.approx(_hot5(T[g.density() > 0]), rel=5e-7)
