"""Launches with few packages: chunks of 64 ids, statistics in slots, and a
rotation over more frequencies than a wave looks at once, some of them
without packages."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bg", [1, 63, 64, 65, 5000])
def test_every_package_is_counted_once(n_bg):
    from paper_1812_06632_amd import soc, workloads as W

    P = W.sphere_problem(n=8, n_packages=n_bg)
    ctx = soc.Context(0)
    g = soc.grid_from_workload(ctx, P.grid)
    f = (float(P.nu[0]), float(P.w[0]), float(P.sigma_abs[0]), float(P.sigma_sca[0]), float(P.g[0]))
    A = torch.zeros(P.grid.ncells, dtype=torch.float64, device="cuda")
    for _ in range(2):
        A.zero_()
        st = soc.simulate_frequency(ctx, g, f, A, I_bg=float(P.I_bg[0]), n_bg=n_bg, seed=3, stats=True)
        assert st["packages"] == n_bg
        assert abs(float(A.sum()) + st["e_escaped"] - st["e_emitted"]) <= 1e-9 * st["e_emitted"]
    total = ctx.read_stats(reset=True)
    assert total["packages"] == 2 * n_bg and ctx.read_stats()["packages"] == 0


@pytest.mark.parametrize("spread", [0, 1])
def test_rotation_over_many_frequencies(spread):
    from paper_1812_06632_amd import soc, workloads as W

    K = 130
    P = W.lognormal_problem(n=8, K=K)
    ctx = soc.Context(0)
    ctx.set_option("multi_spread", spread)
    g = soc.grid_from_workload(ctx, P.grid)
    freqs = [(float(P.nu[k]), float(P.w[k]), float(P.sigma_abs[k]), float(P.sigma_sca[k]), float(P.g[k])) for k in range(K)]
    counts = [0 if k < 66 or k % 7 == 0 else 40 + k for k in range(K)]
    src = [dict(I_bg=float(P.I_bg[k]), n_bg=counts[k]) for k in range(K)]
    A = torch.zeros(P.grid.ncells, dtype=torch.float64, device="cuda")
    B = torch.zeros_like(A)
    st = soc.simulate_frequencies(ctx, g, freqs, A, src, range(K), seed=5, iteration=1, stats=True)
    steps = 0
    for k in range(K):
        one = soc.simulate_frequency(ctx, g, freqs[k], B, seed=5, iteration=1, freq_index=k, stats=True, **src[k])
        steps += one["cell_steps"]
    assert st["packages"] == sum(counts) and st["cell_steps"] == steps
    # the same FP64 deposits in another order
    np.testing.assert_allclose(A.cpu().numpy(), B.cpu().numpy(), rtol=1e-11)


@pytest.mark.parametrize("n_bg", [1, 4095, 4097, 20000])
@pytest.mark.parametrize("lds", [0, 13824])
def test_batch_items_cover_every_id(n_bg, lds):
    """Pairs cut into several LDS items or small tiles add up to the single
    calls."""
    from paper_1812_06632_amd import soc, workloads as W

    ctx = soc.Context(0)
    ctx.set_option("batch_lds_cells", lds)
    grids, (nu, w, sabs, ssca, hg, I), _ = W.batch_clouds(n_models=3, K=2, n_min=8, n_max=16)
    G = [soc.grid_from_workload(ctx, g) for g in grids]
    f = [(float(nu[k]), float(w[k]), float(sabs[k]), float(ssca[k]), float(hg[k])) for k in range(2)]
    A = [torch.zeros(g.ncells, dtype=torch.float64, device="cuda") for g in G]
    pairs = [dict(grid=m, freq=f[k], freq_index=k, absorbed=A[m], I_bg=float(I[k]), n_bg=n_bg) for m in range(3) for k in range(2)]
    b = soc.Batch(ctx, G, pairs, seed=11)
    assert b.info()[1] == 6 * n_bg
    st = b.run(iteration=2, stats=True)
    assert st["packages"] == 6 * n_bg
    steps = 0
    for m in range(3):
        B = torch.zeros_like(A[m])
        for k in range(2):
            steps += soc.simulate_frequency(ctx, G[m], f[k], B, I_bg=float(I[k]), n_bg=n_bg, seed=11 ^ (m << 32), iteration=2,
                                            freq_index=k, stats=True)["cell_steps"]
        # the same FP64 deposits in another order
        np.testing.assert_allclose(A[m].cpu().numpy(), B.cpu().numpy(), rtol=1e-11)
    assert st["cell_steps"] == steps


@pytest.mark.parametrize("n_dark", [2**31 - 500, 2**31, 2**32 - 1 - 1000])
@pytest.mark.parametrize("lds", [0, 13824])
def test_batch_ids_beyond_31_bits(n_dark, lds):
    """A pair's last packages, those of a source, have ids on both sides of
    2^31 and up to 2^32 - 2; the ids before them carry no energy (counted,
    not traced)."""
    from paper_1812_06632_amd import soc, workloads as W

    P = W.sphere_problem(n=8, n_packages=1000)
    ctx = soc.Context(0)
    ctx.set_option("batch_lds_cells", lds)
    g = soc.grid_from_workload(ctx, P.grid)
    f = (float(P.nu[0]), float(P.w[0]), float(P.sigma_abs[0]), float(P.sigma_sca[0]), float(P.g[0]))
    src = dict(ps_pos=[[3.5, 4.25, 4.5]], ps_Lnu=[1e20], n_ps_pk=1000)
    A = torch.zeros(P.grid.ncells, dtype=torch.float64, device="cuda")
    B = torch.zeros_like(A)
    one = soc.simulate_frequency(ctx, g, f, B, seed=11, iteration=2, freq_index=0, stats=True, **src)
    b = soc.Batch(ctx, [g], [dict(grid=0, freq=f, freq_index=0, absorbed=A, n_bg=n_dark, I_bg=0.0, **src)], seed=11)
    st = b.run(iteration=2, stats=True)
    assert st["packages"] == n_dark + 1000
    for key in ("cell_steps", "scatterings", "runaways"):
        assert st[key] == one[key], key
    assert st["e_emitted"] == pytest.approx(one["e_emitted"], rel=1e-12, abs=0)
    # the same FP64 deposits in another order
    np.testing.assert_allclose(A.cpu().numpy(), B.cpu().numpy(), rtol=1e-11)
