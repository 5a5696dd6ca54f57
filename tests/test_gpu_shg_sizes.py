"""The grain solver at the sizes where its tables, tiles and parts change:
frequencies and bins on both sides of 64, the smallest and largest models,
grids below and above one tile of 64 cells, fields so strong that the
unnormalised populations are rescaled."""
import numpy as np
import pytest

from oracle import shg_oracle as O
from paper_1812_06632_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _solve(G, grid, A, populations):
    from paper_1812_06632_amd import soc

    ctx = soc.Context(0)
    g = soc.grid_from_workload(ctx, grid)
    model = soc.ShgModel(ctx, G)
    Ad = torch.from_numpy(A).cuda()
    E = torch.full_like(Ad, -1.0)
    P = torch.full((grid.ncells, len(G.a_cm), G.U.shape[1]), -1.0, dtype=torch.float64, device="cuda") if populations else None
    soc.shg_solve(ctx, g, model, Ad, E, P)
    again = torch.empty_like(E)
    soc.shg_solve(ctx, g, model, Ad, again)
    assert torch.equal(E, again)   # fixed order of every sum, with and without the populations
    return E.cpu().numpy(), P.cpu().numpy() if populations else None


@pytest.mark.parametrize("K,N,S", [(1, 2, 1), (2, 3, 2), (63, 64, 2), (64, 65, 1), (65, 64, 1), (128, 128, 2), (127, 33, 3)])
def test_matches_oracle(K, N, S):
    nu, w = W.frequency_grid(K) if K > 1 else (np.array([3e14]), np.array([1e14]))
    G = W.grain_model(nu, w, n_size=S, n_enthalpy=N)
    rng = np.random.default_rng(K + N)
    rho = rng.uniform(0.5, 2.0, (2, 3, 3)).astype(np.float32)
    rho[1, 1, 1] = 0.0
    grid = W.regular_grid(rho, 1.0e17)
    d = grid.density().astype(np.float64)
    V = np.full(grid.ncells, 1.0e51)
    field = 10 ** rng.uniform(-3.0, 4.0, grid.ncells)
    A = 4 * np.pi * (W.isrf(nu) * G.sigma_per_H * w)[:, None] * (field * d * V)[None, :]
    E_o, P_o = O.shg_solve(G, d, V, A)
    E, P = _solve(G, grid, A, True)
    leaf = d > 0
    # FP64 sums of positive terms; the first bucket's (U + h nu) - U rounds as the oracle's
    np.testing.assert_allclose(P[leaf], P_o[leaf], rtol=1e-9, atol=1e-13)
    np.testing.assert_allclose(E, E_o, rtol=1e-9, atol=1e-12 * np.abs(E_o).max())
    assert not E[:, ~leaf].any() and not P[~leaf].any()


@pytest.mark.parametrize("cells", [1, 15, 17, 63, 65, 1000])
def test_cells_do_not_depend_on_their_neighbours(cells):
    """Every cell of a line equals the same cell in a larger grid, whatever
    tile, wave and size part it falls into."""
    nu, w = W.frequency_grid(40)
    G = W.grain_model(nu, w, n_size=5, n_enthalpy=50)
    rng = np.random.default_rng(2)
    n = 1200
    d = rng.uniform(0.5, 2.0, n).astype(np.float32)
    field = 10 ** rng.uniform(-2.0, 9.0, n)
    A = 4 * np.pi * (W.isrf(nu) * G.sigma_per_H * w)[:, None] * (field * d * 1.0e51)[None, :]
    whole, Pw = _solve(G, W.regular_grid(d.reshape(1, 1, n), 1.0e17), A, True)
    assert np.isfinite(whole).all() and np.isfinite(Pw).all()
    np.testing.assert_allclose(Pw.sum(axis=2), 1.0, rtol=1e-12)
    E, P = _solve(G, W.regular_grid(d[:cells].reshape(1, 1, cells), 1.0e17), np.ascontiguousarray(A[:, :cells]), True)
    np.testing.assert_array_equal(P, Pw[:cells])
    # the size parts of a small grid are added in another grouping
    np.testing.assert_allclose(E, whole[:, :cells], rtol=1e-13)


def _line(n, G, nu, w, seed):
    rng = np.random.default_rng(seed)
    d = rng.uniform(0.5, 2.0, n).astype(np.float32)
    field = 10 ** rng.uniform(-2.0, 4.0, n)
    A = 4 * np.pi * (W.isrf(nu) * G.sigma_per_H * w)[:, None] * (field * d * 1.0e51)[None, :]
    return W.regular_grid(d.reshape(1, 1, n), 1.0e17), A


@pytest.mark.parametrize("external", [False, True])
def test_captured_solve_outlives_larger_ones(external):
    """A graph of a small solve (sizes in parts outside of a capture) replayed
    after larger solves and after solves of other models, with eager work and
    synchronizations between the replays; captured by the library and by the
    caller."""
    from paper_1812_06632_amd import soc

    nu, w = W.frequency_grid(40)
    G = W.grain_model(nu, w, n_size=5, n_enthalpy=50)
    G2 = W.grain_model(nu, w, n_size=9, n_enthalpy=50)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx = soc.Context(0, stream=s)
        small, As = _line(100, G, nu, w, 1)
        large, Al = _line(5000, G, nu, w, 2)
        gs, gl = soc.grid_from_workload(ctx, small), soc.grid_from_workload(ctx, large)
        m, m2 = soc.ShgModel(ctx, G), soc.ShgModel(ctx, G2)
        As, Al = torch.from_numpy(As).cuda(), torch.from_numpy(Al).cuda()
        want, El = torch.empty_like(As), torch.empty_like(Al)
        soc.shg_solve(ctx, gs, m, As, want)
        E = torch.full_like(As, -1.0)
        if external:
            s.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                soc.shg_solve(ctx, gs, m, As, E)
        else:
            soc.graph_begin(ctx)
            soc.shg_solve(ctx, gs, m, As, E)
            g = soc.graph_end(ctx)
        assert torch.all(E == -1.0)   # recorded, not run
        for k in range(4):
            soc.shg_solve(ctx, gl, m, Al, El)
            soc.shg_solve(ctx, gl, m2, Al, El)
            E.fill_(-1.0)
            (g.replay if external else g.launch)()
            soc.shg_solve(ctx, gl, m, Al, El)
            if k % 2:
                s.synchronize()
            # the sum over sizes in one part
            np.testing.assert_allclose(E.cpu().numpy(), want.cpu().numpy(), rtol=1e-13)
        s.synchronize()


def test_solves_on_two_streams_take_turns():
    """One model, two streams, nothing between the solves: the parts of one do
    not reach the other."""
    import ctypes

    from paper_1812_06632_amd import soc

    nu, w = W.frequency_grid(40)
    G = W.grain_model(nu, w, n_size=6, n_enthalpy=50)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    ctx = soc.Context(0, stream=streams[0])
    m = soc.ShgModel(ctx, G)
    work = []
    for n in (3000, 1000):
        grid, A = _line(n, G, nu, w, n)
        A = torch.from_numpy(A).cuda()
        work.append((soc.grid_from_workload(ctx, grid), A, torch.empty_like(A), torch.empty_like(A)))
    torch.cuda.synchronize()
    for g, A, want, _ in work:
        soc.shg_solve(ctx, g, m, A, want)
        torch.cuda.synchronize()
    for _ in range(20):
        for s, (g, A, _, E) in zip(streams, work):
            assert soc._lib.soc_ctx_set_stream(ctx.h, ctypes.c_void_p(s.cuda_stream)) == 0
            soc.shg_solve(ctx, g, m, A, E)
    torch.cuda.synchronize()
    for _, _, want, E in work:
        assert torch.equal(E, want)


@pytest.mark.parametrize("absorbed", [np.nan, np.inf])
def test_sizes_without_grains_absorb_nothing(absorbed):
    """Whatever the field: their grains stay in the lowest bin and emit
    nothing, and the other cells of the wave are not touched."""
    from paper_1812_06632_amd import soc

    nu, w = W.frequency_grid(40)
    G = W.grain_model(nu, w, n_size=3, n_enthalpy=50)
    grid, A = _line(40, G, nu, w, 3)
    A[7, 5] = absorbed

    def solve():   # (as _solve, whose comparison of two solves takes no NaN)
        ctx = soc.Context(0)
        Ad = torch.from_numpy(A).cuda()
        E = torch.full_like(Ad, -1.0)
        P = torch.full((grid.ncells, 3, 50), -1.0, dtype=torch.float64, device="cuda")
        soc.shg_solve(ctx, soc.grid_from_workload(ctx, grid), soc.ShgModel(ctx, G), Ad, E, P)
        return E.cpu().numpy(), P.cpu().numpy()

    G.abundance[1] = 0.0
    E, P = solve()
    assert not np.isfinite(E[:, 5]).any() and not np.isfinite(P[5, [0, 2]]).any()   # two sizes have grains
    np.testing.assert_array_equal(P[:, 1, 0], 1.0)
    assert not P[:, 1, 1:].any()
    others = np.arange(40) != 5
    assert np.isfinite(E[:, others]).all() and np.isfinite(P[others]).all()
    G.abundance[:] = 0.0
    E, P = solve()
    assert not E.any()
    np.testing.assert_array_equal(P[:, :, 0], 1.0)
