"""The performance cases of this framework: what its users run, at the sizes they run it.

A case is a dict of plain values; its "kind" names the path:

  single       one frequency and the temperature solve: the smallest whole calls
  pass         every frequency of an iteration in one call and the temperature solve, on a regular grid or an
               octree, with the constant sources or with the dust emission (optionally with diagonal ALI)
  batch        many clouds of uneven size in one launch, and their temperatures
  scatter      a scattered-light image
  temperature  the temperature solve with the convergence statistics of one iteration
  map          an emission map
  grains       stochastically heated grains: temperature distributions and their emission
  forward      the U-Net's prediction
  gradient     a training batch's loss and parameter gradients

`prepare` builds a case's inputs from a seed, `run` makes one pass through the public entry points, `exact` gives
the outputs in 64 bits from plain torch where the path is deterministic (a Monte Carlo pass has no such value) and
`work` counts what a pass cannot do without.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1812_06632_amd import soc
from paper_1812_06632_amd import workloads as W

T_FLOOR, T_MAX = 2.0, 3000.0
STEP_FLOPS = 60           # arithmetic of one cell step: three face distances, optical depth, absorption, position
BUDGET = 128 * 64 * 1.0e6   # cell crossings of the largest pass, in units of (cells per axis) x frequencies x packages


# ------------------------------------------------------------------ cases
def listed():
    return [
        # the smallest whole calls: one frequency of a small sphere, as in a parameter study of many small models
        {"name": "sphere 16", "kind": "single", "n": 16, "packages": 20000, "noalloc": False},
        # the constant-source pass of the clouds the learned start is trained on
        {"name": "cloud 64 constant", "kind": "pass", "octree": 1, "nx": 64, "ny": 64, "nz": 64, "K": 32,
         "packages": 200000, "dust": False, "ali": False},
        # a dust iteration of the benchmark cloud
        {"name": "cloud 128 dust", "kind": "pass", "octree": 1, "nx": 128, "ny": 128, "nz": 128, "K": 64,
         "packages": 1000000, "dust": True, "ali": False},
        # a cut-out of a cloud with odd edges, few packages, accelerated iteration
        {"name": "cut-out dust ALI", "kind": "pass", "octree": 1, "nx": 45, "ny": 61, "nz": 38, "K": 16,
         "packages": 100000, "dust": True, "ali": True},
        # a refined cloud with a source in its core
        {"name": "octree constant", "kind": "pass", "octree": 3, "nx": 32, "ny": 32, "nz": 32, "K": 32,
         "packages": 200000, "dust": False, "ali": False},
        # uneven small and middle-sized models together: a grid of models
        {"name": "batch of 24", "kind": "batch", "models": 24, "n_min": 16, "n_max": 72, "K": 8, "packages": 30000},
        # an image of scattered light at optical wavelengths
        {"name": "scatter 128", "kind": "scatter", "n": 128, "packages": 1000000, "forced": True, "direct": True,
         "axis": 2},
        # the solve and the stopping rule's statistics after every iteration
        {"name": "temperature 128", "kind": "temperature", "n": 128, "K": 64},
        # a far-infrared map of a refined cloud
        {"name": "map octree", "kind": "map", "octree": 3, "n": 32, "axis": 0},
        # the paper's grain model (25 sizes, 128 bins, 128 frequencies)
        {"name": "grains 32", "kind": "grains", "n": 32, "S": 25, "N": 128, "K": 128, "populations": False},
        # the learned start of one cloud
        {"name": "unet forward", "kind": "forward", "side": 64, "batch": 1, "base": 32, "levels": 4},
        # one training batch
        {"name": "unet gradient", "kind": "gradient", "side": 64, "batch": 4, "base": 32, "levels": 4},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["single", "pass", "pass", "octree", "batch", "scatter", "temperature", "map", "grains",
                       "forward", "gradient"])
    if kind == "single":
        return {"kind": kind, "n": rng.randint(8, 32), "packages": int(_log(rng, 1e4, 1e5)),
                "noalloc": rng.random() < 0.5}
    if kind == "pass":
        n = [int(_log(rng, 16, 128)) for _ in range(3)]
        K = int(_log(rng, 4, 64))
        return {"kind": kind, "octree": 1, "nx": n[0], "ny": n[1], "nz": n[2], "K": K,
                "packages": int(_log(rng, 2e4, min(1e6, BUDGET / (max(n) * K)))), "dust": rng.random() < 0.6,
                "ali": rng.random() < 0.3}
    if kind == "octree":
        n, levels, K = int(_log(rng, 8, 32)), rng.randint(2, 3), int(_log(rng, 4, 32))
        return {"kind": "pass", "octree": levels, "nx": n, "ny": n, "nz": n, "K": K,
                "packages": int(_log(rng, 2e4, 4e5)), "dust": rng.random() < 0.5, "ali": False}
    if kind == "batch":
        return {"kind": kind, "models": rng.randint(4, 32), "n_min": 16, "n_max": 8 * rng.randint(3, 10),
                "K": rng.randint(2, 12), "packages": int(_log(rng, 1e4, 1e5))}
    if kind == "scatter":
        return {"kind": kind, "n": int(_log(rng, 24, 128)), "packages": int(_log(rng, 1e5, 1e6)),
                "forced": rng.random() < 0.7, "direct": rng.random() < 0.5, "axis": rng.choice([0, 1, 2, 4, 5, 6])}
    if kind == "temperature":
        return {"kind": kind, "n": int(_log(rng, 16, 160)), "K": int(_log(rng, 16, 128))}
    if kind == "map":
        octree = rng.randint(1, 3)
        return {"kind": kind, "octree": octree, "n": int(_log(rng, 12, 128 >> (octree - 1))),
                "axis": rng.choice([0, 1, 2, 4, 5, 6])}
    if kind == "grains":
        S, N, K = rng.randint(4, 25), rng.randint(32, 128), rng.randint(24, 128)
        n = min(40, int((3.0e6 * 128 * 128 / (S * N * K)) ** (1 / 3)))
        return {"kind": kind, "n": int(_log(rng, 8, n)), "S": S, "N": N, "K": K, "populations": rng.random() < 0.3}
    levels = rng.randint(2, 4)
    step = 1 << (levels - 1)
    side = step * max(2, int(_log(rng, 16, 64)) // step)
    return {"kind": kind, "side": side, "batch": rng.randint(1, 4), "base": rng.choice([16, 32]), "levels": levels}


# ------------------------------------------------------------------ inputs
_ctx = None


def _context():
    """The program's library context: one for all its calls."""
    global _ctx
    if _ctx is None:
        _ctx = soc.Context(0)
    return _ctx


def _cloud(nx, ny, nz, seed, sources=True, sigma_ln=1.0, tau=5.0):
    """A lognormal cloud of any shape (cut from a cube) and its two sources, whose cells are empty."""
    n = max(nx, ny, nz)
    rho = W.grf_lognormal(n, sigma_ln, seed)[:nz, :ny, :nx]
    cell = W.PC_CM / n
    rho = rho * (tau / (W.SIGMA_V * W.PC_CM * rho.mean()))
    pos = np.array([[math.floor(f * m) + 0.5 for f, m in zip(fr, (nx, ny, nz))]
                    for fr in ((0.3, 0.5, 0.5), (0.7, 0.5, 0.5))]) if sources else np.zeros((0, 3))
    for p in pos:
        rho[int(p[2]), int(p[1]), int(p[0])] = 0.0
    return W.regular_grid(rho.astype(np.float32), cell), pos


def _dust(K):
    nu, w = W.frequency_grid(K)
    sabs, ssca, g = W.dust_model(nu)
    return nu, w, sabs, ssca, g, W.isrf(nu)


def _freqs(nu, w, sabs, ssca, g):
    return [tuple(float(v) for v in f) for f in zip(nu, w, sabs, ssca, g)]


def _centres(g):
    """Cell centres (root units) and edges of every cell of a grid."""
    lo = np.empty((g.ncells, 3))
    edge = np.empty(g.ncells)
    c = np.arange(g.nroot)
    lo[:g.nroot] = np.stack([c % g.nx, (c // g.nx) % g.ny, c // (g.nx * g.ny)], axis=1)
    edge[:g.nroot] = 1.0
    words = g.words.view(np.int32)
    o = np.arange(8)
    step = np.stack([o & 1, (o >> 1) & 1, (o >> 2) & 1], axis=1)
    for L in range(g.nlevels - 1):
        cells = np.arange(g.level_offset[L], g.level_offset[L + 1])
        cells = cells[words[cells] < 0]
        kids = (-words[cells].astype(np.int64))[:, None] + o
        edge[kids] = 0.5 ** (L + 1)
        lo[kids] = lo[cells][:, None, :] + 0.5 ** (L + 1) * step
    return lo + 0.5 * edge[:, None], edge


def _temperatures(g, pos, seed):
    """A dust temperature field like a solved one: about 17 K in the external field, hotter towards the sources, a few
    per cent of scatter; 0 in empty and refined cells."""
    rng = np.random.default_rng(seed + 77)
    x, _ = _centres(g)
    heat = np.ones(g.ncells)
    for p in pos:
        heat += 2.0e5 / (((x - p) ** 2).sum(axis=1) * (128.0 / max(g.nx, g.ny, g.nz)) ** 2 + 0.25)
    T = 17.0 * heat ** (1 / 5.8) * np.exp(0.03 * rng.standard_normal(g.ncells))
    return np.where(g.density() > 0, np.minimum(T, 1500.0), 0.0).astype(np.float32)


def _octree(n_root, levels, seed):
    """A refined lognormal cloud with a dense core; the seed varies the densities of its cells, not the refinement."""
    g = W.octree_lognormal(n_root=n_root, nlevels=levels)
    _vary(g, seed, 0.3)
    return g


def _vary(g, seed, scatter):
    leaf = ~g.is_link()
    rho = g.words.view(np.float32)
    rng = np.random.default_rng(seed + 21)
    rho[leaf] *= np.exp(rng.normal(0.0, scatter) + scatter * rng.standard_normal(int(leaf.sum()))).astype(np.float32)


def _rng_seed(seed):
    return 1 + (int(seed) * 2654435761) % (1 << 31)


def prepare(case, seed):
    ctx = _context()
    return globals()["_prepare_" + case["kind"]](case, int(seed), ctx)


def _table(ctx, nu, w, sabs):
    return soc.temp_table_build(ctx, nu, w, sabs, T_FLOOR, T_MAX, 4096)


def _prepare_single(case, seed, ctx):
    P = W.sphere_problem(n=case["n"], n_packages=case["packages"], tau_centre_edge=0.5 + (seed % 7) * 0.25)
    grid = soc.grid_from_workload(ctx, P.grid)
    return {"case": case, "ctx": ctx, "grid": grid, "seed": _rng_seed(seed),
            "freq": _freqs(P.nu, P.w, P.sigma_abs, P.sigma_sca, P.g)[0], "I": float(P.I_bg[0]), "n": P.n_bg,
            "table": _table(ctx, P.emit_nu, P.emit_w, P.emit_sigma_abs),
            "A": torch.zeros(grid.ncells, dtype=torch.float64, device="cuda"),
            "T": torch.zeros(grid.ncells, dtype=torch.float32, device="cuda")}


def _prepare_pass(case, seed, ctx):
    nx, ny, nz, K, n = (case[k] for k in ("nx", "ny", "nz", "K", "packages"))
    if case["octree"] > 1:
        g = _octree(nx, case["octree"], seed)
        pos = np.full((1, 3), 0.5 * nx) + 0.01
    else:
        g, pos = _cloud(nx, ny, nz, seed)
    nu, w, sabs, ssca, hg, I = _dust(K)
    grid = soc.grid_from_workload(ctx, g)
    cells = grid.ncells
    state = {"case": case, "ctx": ctx, "grid": grid, "seed": _rng_seed(seed), "freqs": _freqs(nu, w, sabs, ssca, hg),
             "table": _table(ctx, nu, w, sabs), "A": torch.zeros(cells, dtype=torch.float64, device="cuda"),
             "T": torch.zeros(cells, dtype=torch.float32, device="cuda"), "A0": None, "self": None, "emitted": None}
    if case["dust"]:
        # what the constant sources gave and the temperatures of the iteration before
        T = _temperatures(g, pos, seed)
        state["T_old"] = torch.from_numpy(T).cuda()
        kept = np.random.default_rng(seed + 5).uniform(0.5, 1.5, cells) * g.density() * 1e-30 * g.root_cell_cm ** 3
        state["A0"] = torch.from_numpy(kept).cuda()
        src = {"T": state["T_old"], "n_dust": n, "dust_mode": 1}
        if case["ali"]:
            state["self"], state["emitted"] = (torch.zeros(cells, dtype=torch.float64, device="cuda") for _ in "ab")
            src |= {"ali_self": state["self"], "ali_emitted": state["emitted"]}
        state["sources"] = [src] * K
    else:
        L = W.blackbody_Lnu(nu, 1.0e6 * W.L_SUN, 1.0e4)
        state["sources"] = [{"I_bg": float(I[k]), "ps_pos": pos, "ps_Lnu": [float(L[k])] * len(pos), "n_bg": n // 2,
                             "n_ps_pk": max(1, n // 2 // len(pos))} for k in range(K)]
        state["T_old"] = None
    return state


def _prepare_batch(case, seed, ctx):
    grids, (nu, w, sabs, ssca, hg, I), packages = W.batch_clouds(
        n_models=case["models"], K=case["K"], n_min=case["n_min"], n_max=case["n_max"],
        pk_min=case["packages"] / 3, pk_max=case["packages"] * 3)
    for m, g in enumerate(grids):
        _vary(g, 100 * seed + m, 0.3)
    freqs = _freqs(nu, w, sabs, ssca, hg)
    built = [soc.grid_from_workload(ctx, g) for g in grids]
    A = torch.zeros(sum(g.ncells for g in grids), dtype=torch.float64, device="cuda")
    T = torch.zeros(A.numel(), dtype=torch.float32, device="cuda")
    cut = [0] + list(np.cumsum([g.ncells for g in grids]))
    parts = [(A[a:b], T[a:b]) for a, b in zip(cut, cut[1:])]
    pairs = [{"grid": m, "freq": freqs[k], "freq_index": k, "absorbed": parts[m][0], "I_bg": float(I[k]),
              "n_bg": int(packages[m, k])} for m in range(case["models"]) for k in range(case["K"])]
    return {"case": case, "ctx": ctx, "grids": built, "A": A, "T": T, "parts": parts, "table": _table(ctx, nu, w, sabs),
            "batch": soc.Batch(ctx, built, pairs, seed=_rng_seed(seed))}


def _prepare_scatter(case, seed, ctx):
    n = case["n"]
    g, pos = _cloud(n, n, n, seed)
    nu = np.array([2.99792458e10 / 0.55e-4])
    sabs, ssca, hg = W.dust_model(nu)
    L = W.blackbody_Lnu(nu, 1.0e6 * W.L_SUN, 1.0e4)
    grid = soc.grid_from_workload(ctx, g)
    shape = soc.scatter_image_shape(grid, case["axis"])
    return {"case": case, "ctx": ctx, "grid": grid, "seed": _rng_seed(seed), "pos": pos, "L": [float(L[0])] * len(pos),
            "freq": _freqs(nu, [1.0e14], sabs, ssca, hg)[0], "I": float(W.isrf(nu)[0]),
            "image": torch.zeros(shape, dtype=torch.float64, device="cuda")}


def _planck(nu, T):
    """B_nu(T) in 64 bits (cgs), torch tensors."""
    x = 6.62607015e-27 * nu / (1.380649e-16 * T)
    return 2.0 * 6.62607015e-27 * nu ** 3 / 2.99792458e10 ** 2 / torch.expm1(torch.clamp(x, max=700.0))


def _gamma(T, nu, w, sabs):
    """4 pi sum_k w_k sigma_k B_nu_k(T)."""
    out = torch.zeros_like(T)
    for a, b, c in zip(nu.tolist(), w.tolist(), sabs.tolist()):
        out += 4.0 * math.pi * b * c * _planck(a, T)
    return out


def _temperature_inputs(case, seed):
    n = case["n"]
    g, pos = _cloud(n, n, n, seed)
    nu, w, sabs, *_ = _dust(case["K"])
    rng = np.random.default_rng(seed + 3)
    T = _temperatures(g, pos, seed)
    true = torch.from_numpy(np.maximum(T, 1.0) * np.exp(0.02 * rng.standard_normal(g.ncells))).double().cuda()
    A = _gamma(true, nu, w, sabs) * torch.from_numpy(g.density()).double().cuda() * g.root_cell_cm ** 3
    A[torch.from_numpy(rng.random(g.ncells) < 0.001).cuda()] = 0.0   # cells no package reached
    return g, (nu, w, sabs), A, torch.from_numpy(T).cuda()


def _prepare_temperature(case, seed, ctx):
    g, model, A, T = _temperature_inputs(case, seed)
    return {"case": case, "ctx": ctx, "grid": soc.grid_from_workload(ctx, g), "table": _table(ctx, *model), "A": A,
            "T_old": T, "T": torch.zeros_like(T)}


def _map_inputs(case, seed):
    n = case["n"]
    if case["octree"] > 1:
        g, pos = _octree(n, case["octree"], seed), np.full((1, 3), 0.5 * n)
    else:
        g, pos = _cloud(n, n, n, seed)
    nu = np.array([2.99792458e10 / 100e-4])
    sabs, ssca, hg = W.dust_model(nu)
    return g, _temperatures(g, pos, seed), _freqs(nu, [1.0e11], sabs, ssca, hg)[0]


def _prepare_map(case, seed, ctx):
    g, T, freq = _map_inputs(case, seed)
    grid = soc.grid_from_workload(ctx, g)
    return {"case": case, "ctx": ctx, "grid": grid, "freq": freq, "T": torch.from_numpy(T).cuda(),
            "image": torch.empty(soc.map_shape(grid, case["axis"]), dtype=torch.float32, device="cuda")}


def _grain_inputs(case, seed):
    """Absorbed energies per band of cells between a tenth and a hundred times the external field, reddened."""
    n, K = case["n"], case["K"]
    g, _ = _cloud(n, n, n, seed, sources=False)
    nu, w = W.frequency_grid(K)
    G = W.grain_model(nu, w, n_size=case["S"], n_enthalpy=case["N"])
    rng = np.random.default_rng(seed + 9)
    dens = torch.from_numpy(g.density()).double().cuda()
    field = torch.from_numpy(np.exp(rng.normal(0.7, 1.2, g.ncells))).cuda()
    tau = torch.from_numpy(np.exp(rng.normal(-0.5, 0.8, g.ncells))).cuda()
    per_H = torch.from_numpy(G.sigma_per_H * W.isrf(nu) * w * 4.0 * math.pi).cuda()
    red = torch.from_numpy(nu / (2.99792458e10 / 0.55e-4)).cuda()
    A = per_H[:, None] * torch.exp(-red[:, None] * tau) * (field * dens * g.root_cell_cm ** 3)
    return g, G, A.contiguous()


def _prepare_grains(case, seed, ctx):
    g, G, A = _grain_inputs(case, seed)
    P = torch.empty((g.ncells, case["S"], case["N"]), dtype=torch.float64, device="cuda") if case["populations"] else None
    return {"case": case, "ctx": ctx, "grid": soc.grid_from_workload(ctx, g), "model": soc.ShgModel(ctx, G), "A": A,
            "E": torch.empty_like(A), "P": P}


CIN, COUT = 4, 2   # features and targets of the learned start


def _unet_layers(base, levels):
    """(kind, input channels, output channels) of every layer, in parameter order."""
    ch = [base << l for l in range(levels)]
    out, c = [], CIN
    for l in range(levels):
        out += [("conv", c, ch[l]), ("conv", ch[l], ch[l])]
        if l < levels - 1:
            out.append(("down", ch[l], ch[l + 1]))
            c = ch[l + 1]
    for l in range(levels - 2, -1, -1):
        out += [("up", ch[l + 1], ch[l]), ("conv", 2 * ch[l], ch[l]), ("conv", ch[l], ch[l])]
    return out + [("conv", ch[0], COUT)]


def _unet_inputs(case, seed):
    """Parameters (He-normal weights, small biases), feature-like smooth fields and a target."""
    gen = torch.Generator().manual_seed(seed)
    params = []
    for kind, ci, co in _unet_layers(case["base"], case["levels"]):
        taps = 27 if kind == "conv" else 8
        params += [torch.randn(taps * ci * co, generator=gen) * math.sqrt(2.0 / (taps * ci)),
                   0.02 * torch.randn(co, generator=gen)]
    s, b = case["side"], case["batch"]
    coarse = torch.randn((b, CIN + COUT, 6, 6, 6), generator=gen).cuda()
    fine = torch.nn.functional.interpolate(coarse, size=(s, s, s), mode="trilinear", align_corners=False)
    fine = (0.6 * fine + 0.1 * torch.randn(fine.shape, generator=gen).cuda()).permute(0, 2, 3, 4, 1)
    return torch.cat(params), fine[..., :CIN].contiguous(), fine[..., CIN:].contiguous()


def _prepare_forward(case, seed, ctx):
    params, x, t = _unet_inputs(case, seed)
    s = case["side"]
    net = soc.UNet(ctx, CIN, COUT, case["base"], case["levels"], case["batch"], (s, s, s), seed=seed)
    net.set_params(params.numpy())
    return {"case": case, "ctx": ctx, "net": net, "x": x, "t": t, "y": torch.empty_like(t)}


_prepare_gradient = _prepare_forward


# ------------------------------------------------------------------ passes
def run(state):
    return globals()["_run_" + state["case"]["kind"]](state)


def _run_single(s):
    s["A"].zero_()
    soc.simulate_frequency(s["ctx"], s["grid"], s["freq"], s["A"], I_bg=s["I"], n_bg=s["n"], seed=s["seed"],
                           noalloc=s["case"]["noalloc"])
    soc.update_temperature(s["ctx"], s["grid"], s["table"], s["A"], s["T"])
    return {"A": s["A"], "T": s["T"]}


def _run_pass(s):
    if s["A0"] is None:
        s["A"].zero_()
    else:
        s["A"].copy_(s["A0"])
    if s["self"] is not None:
        s["self"].zero_()
        s["emitted"].zero_()
    soc.simulate_frequencies(s["ctx"], s["grid"], s["freqs"], s["A"], s["sources"], range(len(s["freqs"])),
                             seed=s["seed"], iteration=2)
    stats = soc.update_temperature(s["ctx"], s["grid"], s["table"], s["A"], s["T"], s["T_old"], stats=True,
                                   ali_self=s["self"], ali_emitted=s["emitted"])
    out = {"A": s["A"], "T": s["T"], "mean": stats["mean_T"], "hot": stats["hot5_mean_T"]}
    if s["self"] is not None:
        out |= {"self": s["self"], "emitted": s["emitted"]}
    return out


def _run_batch(s):
    s["A"].zero_()
    s["batch"].run(iteration=1)
    for grid, (A, T) in zip(s["grids"], s["parts"]):
        soc.update_temperature(s["ctx"], grid, s["table"], A, T)
    return {"A": s["A"], "T": s["T"]}


def _run_scatter(s):
    c = s["case"]
    s["image"].zero_()
    soc.scatter_map(s["ctx"], s["grid"], s["freq"], s["image"], axis=c["axis"], forced=c["forced"], direct=c["direct"],
                    I_bg=s["I"], ps_pos=s["pos"], ps_Lnu=s["L"], n_bg=c["packages"] // 2,
                    n_ps_pk=c["packages"] // 2 // len(s["pos"]), seed=s["seed"])
    return s["image"]


def _run_temperature(s):
    stats = soc.update_temperature(s["ctx"], s["grid"], s["table"], s["A"], s["T"], s["T_old"], stats=True)
    return {"T": s["T"], **stats}


def _run_map(s):
    return soc.map_image(s["ctx"], s["grid"], s["freq"], s["T"], s["case"]["axis"], s["image"])


def _run_grains(s):
    soc.shg_solve(s["ctx"], s["grid"], s["model"], s["A"], s["E"], s["P"])
    return [s["E"]] if s["P"] is None else [s["E"], s["P"]]


def _run_forward(s):
    return s["net"].forward(s["x"], s["y"])


def _run_gradient(s):
    y = s["net"].forward(s["x"], s["y"])
    loss, dy = s["net"].mse(y, s["t"])
    s["net"].backward(dy)
    return {"y": y, "loss": loss, "dy": dy, "gradients": s["net"].get_grads()}


# ------------------------------------------------------------------ work
def work(case):
    kind = case["kind"]
    if kind in ("single", "scatter"):
        n = case["n"]
        cells = n ** 3
        moved = 4 * cells + (20 * cells if kind == "single" else 16 * n * n)
        return {"bytes": moved, "flops": STEP_FLOPS * case["packages"] * n}
    if kind == "pass":
        n = [case[k] << (case["octree"] - 1) for k in ("nx", "ny", "nz")]
        cells = case["nx"] * case["ny"] * case["nz"] * (3 if case["octree"] > 1 else 1)
        moved = cells * (4 + 16 + 4 + (4 + 8 if case["dust"] else 0) + (32 if case["ali"] and case["dust"] else 0))
        return {"bytes": moved, "flops": STEP_FLOPS * case["packages"] * case["K"] * sum(n) / 4}
    if kind == "batch":
        n = (case["n_min"] + case["n_max"]) / 2
        return {"bytes": case["models"] * n ** 3 * 24,
                "flops": STEP_FLOPS * case["models"] * case["K"] * case["packages"] * n}
    if kind == "temperature":
        return {"bytes": 20 * case["n"] ** 3, "flops": 60 * case["n"] ** 3}
    if kind == "map":
        fine = case["n"] << (case["octree"] - 1)
        return {"bytes": 8 * case["n"] ** 3 * (3 if case["octree"] > 1 else 1) + 4 * fine * fine,
                "flops": 40 * case["n"] ** 3}
    if kind == "grains":
        cells, S, N, K = case["n"] ** 3, case["S"], case["N"], case["K"]
        return {"bytes": cells * (16 * K + 4 + (8 * S * N if case["populations"] else 0)),
                "flops": cells * S * (2.0 * N * K + 2.0 * N * N)}
    pos, flops, weights, level, up = case["batch"] * case["side"] ** 3, 0.0, 0, 0, False
    for k, ci, co in _unet_layers(case["base"], case["levels"]):
        if k == "down":
            level += 1
        elif k == "up":
            level -= 1
        taps = {"conv": 27, "down": 8, "up": 1}[k]
        flops += 2.0 * pos / 8 ** level * taps * ci * co
        weights += (27 if k == "conv" else 8) * ci * co + co
    back = kind == "gradient"
    return {"bytes": pos * 4 * (CIN + COUT * (3 if back else 1)) + 4 * weights * (2 if back else 1),
            "flops": flops * (3 if back else 1)}


# ------------------------------------------------------------------ 64 bits
def exact(case, seed):
    """The outputs of `run` in 64 bits, or None for the Monte Carlo paths."""
    f = globals().get("_exact_" + case["kind"])
    return f(case, int(seed)) if f else None


def _exact_temperature(case, seed):
    g, (nu, w, sabs), A, T_old = _temperature_inputs(case, seed)
    dens = torch.from_numpy(g.density()).double().cuda()
    y = A / (dens * g.root_cell_cm ** 3).clamp(min=1e-300)
    lo, hi = torch.full_like(y, math.log(T_FLOOR)), torch.full_like(y, math.log(T_MAX))
    for _ in range(52):
        mid = 0.5 * (lo + hi)
        above = _gamma(torch.exp(mid), nu, w, sabs) > y
        lo, hi = torch.where(above, lo, mid), torch.where(above, mid, hi)
    T = torch.where(dens > 0, torch.exp(0.5 * (lo + hi)), torch.zeros_like(y))
    ends = _gamma(torch.tensor([T_FLOOR, T_MAX], dtype=torch.float64, device="cuda"), nu, w, sabs)
    leaf = dens > 0
    clamped = leaf & ((y <= ends[0]) | (y >= ends[1]))
    T = torch.where(leaf & (y <= ends[0]), torch.full_like(T, T_FLOOR), T)
    v = T[leaf]
    k = math.ceil(0.05 * v.numel())
    was = T_old.double()
    rel = ((T - was).abs() / was)[leaf & (was > 0)]
    return {"T": T, "mean_T": float(v.mean()), "hot5_mean_T": float(torch.topk(v, k).values.mean()),
            "mean_rel_change": float(rel.mean()), "clamped": int(clamped.sum())}


def _exact_map(case, seed):
    g, T, (nu, _, sabs, ssca, _) = _map_inputs(case, seed)
    fine = case["n"] << (case["octree"] - 1)
    # every leaf written over the finest cells it covers: a ray's integral does not change
    dens, temp = torch.zeros((2, fine, fine, fine), dtype=torch.float64, device="cuda")
    x, edge = _centres(g)
    words, rho = g.words.view(np.int32), g.density()
    for L in range(g.nlevels):
        cells = np.arange(g.level_offset[L], g.level_offset[L + 1])
        cells = cells[words[cells] >= 0]
        m = 1 << (case["octree"] - 1 - L)
        at = torch.from_numpy(np.rint((x[cells] - 0.5 * edge[cells][:, None]) * (1 << (case["octree"] - 1))).astype(np.int64)).cuda()
        for dz in range(m):
            for dy in range(m):
                for dx in range(m):
                    i = (at[:, 2] + dz, at[:, 1] + dy, at[:, 0] + dx)
                    dens[i] = torch.from_numpy(rho[cells]).double().cuda()
                    temp[i] = torch.from_numpy(T[cells]).double().cuda()
    ax = 2 - (case["axis"] & 3)   # the arrays are (z, y, x)
    if not case["axis"] & 4:
        dens, temp = dens.flip(ax), temp.flip(ax)   # the observer's side first
    dtau = (sabs + ssca) * dens * (g.root_cell_cm / (1 << (case["octree"] - 1)))
    front = torch.cumsum(dtau, dim=ax) - dtau
    S = torch.where(temp > 0, sabs / (sabs + ssca) * _planck(nu, temp.clamp(min=0.1)), torch.zeros_like(temp))
    return (S * -torch.expm1(-dtau) * torch.exp(-front)).sum(dim=ax)


def _exact_grains(case, seed):
    g, G, A = _grain_inputs(case, seed)
    h = 6.62607015e-27
    dev = {k: torch.from_numpy(np.ascontiguousarray(getattr(G, k))).cuda() for k in ("nu", "w", "abundance", "sigma", "U", "T")}
    nhv = torch.from_numpy(g.density()).double().cuda() * g.root_cell_cm ** 3
    hnu = h * dev["nu"]
    total = (dev["abundance"][:, None] * dev["sigma"]).sum(dim=0)
    E = torch.zeros_like(A)
    N = case["N"]
    pops = torch.empty((g.ncells, case["S"], N), dtype=torch.float64, device="cuda") if case["populations"] else None
    for s in range(case["S"]):
        U, ab = dev["U"][s], dev["abundance"][s]
        grains = ab * nhv
        r = (A * (ab * dev["sigma"][s] / total / hnu)[:, None] / grains).t().contiguous()
        emit = 4.0 * math.pi * dev["sigma"][s] * _planck(dev["nu"][None, :], dev["T"][s][:, None])
        power = (emit * dev["w"]).sum(dim=1)
        P = torch.zeros((g.ncells, N), dtype=torch.float64, device="cuda")
        P[:, 0] = 1.0
        for j in range(1, N):
            part = (((U[:j, None] - U[j - 1]) + hnu[None, :]) / (U[j] - U[j - 1])).clamp(0.0, 1.0)
            v = (P[:, :j] * (r @ part.t())).sum(dim=1) * ((U[j] - U[j - 1]) / power[j])
            big = torch.where(v > 1e200, torch.full_like(v, 1e-200), torch.ones_like(v))
            P = P * big[:, None]
            P[:, j] = v * big
        P = P / P.sum(dim=1, keepdim=True)
        E += ((P * grains[:, None]) @ emit).t()
        if pops is not None:
            pops[:, s] = P
    return [E] if pops is None else [E, pops]


def _conv(h, wt, b, taps):
    """3^3 convolution of one sample [z, y, x, c] with zero padding, or 2^3 with stride 2, as products over taps."""
    n = h.shape[0]
    if taps == 27:
        p = torch.nn.functional.pad(h, (0, 0, 1, 1, 1, 1, 1, 1))
        views = [p[z:z + n, y:y + n, x:x + n] for z in range(3) for y in range(3) for x in range(3)]
    else:
        views = [h[z::2, y::2, x::2] for z in range(2) for y in range(2) for x in range(2)]
    m = views[0].shape[0]
    out = sum(v.reshape(m ** 3, -1) @ wt[t] for t, v in enumerate(views)) + b
    return out.reshape(m, m, m, -1)


def _unet64(params, x, case):
    """The network's prediction for one sample in 64 bits."""
    leak = torch.nn.functional.leaky_relu
    layers, at = iter(_unet_layers(case["base"], case["levels"])), 0

    def layer():
        nonlocal at
        kind, ci, co = next(layers)
        taps = 27 if kind == "conv" else 8
        wt = params[at:at + taps * ci * co].reshape(taps, ci, co)
        b = params[at + taps * ci * co:at + taps * ci * co + co]
        at += taps * ci * co + co
        return taps, wt, b

    def conv(h):
        taps, wt, b = layer()
        return _conv(h, wt, b, taps)

    h, skips = x, []
    for l in range(case["levels"]):
        h = leak(conv(leak(conv(h), 0.1)), 0.1)
        if l < case["levels"] - 1:
            skips.append(h)
            h = leak(conv(h), 0.1)
    for l in range(case["levels"] - 1):
        _, wt, b = layer()
        n = h.shape[0]
        up = torch.stack([h.reshape(n ** 3, -1) @ wt[t] + b for t in range(8)], dim=1)
        up = up.reshape(n, n, n, 2, 2, 2, -1).permute(0, 3, 1, 4, 2, 5, 6).reshape(2 * n, 2 * n, 2 * n, -1)
        h = torch.cat([skips.pop(), leak(up, 0.1)], dim=3)
        h = leak(conv(leak(conv(h), 0.1)), 0.1)
    return conv(h)


def _exact_forward(case, seed):
    params, x, _ = _unet_inputs(case, seed)
    p = params.double().cuda()
    with torch.no_grad():
        return torch.stack([_unet64(p, x[i].double(), case) for i in range(case["batch"])])


def _exact_gradient(case, seed):
    params, x, t = _unet_inputs(case, seed)
    p = params.double().cuda().requires_grad_(True)
    out, loss = [], 0.0
    for i in range(case["batch"]):
        y = _unet64(p, x[i].double(), case)
        part = ((y - t[i].double()) ** 2).sum() / t.numel()
        part.backward()
        out.append(y.detach())
        loss += float(part.detach())
    y = torch.stack(out)
    return {"y": y, "loss": loss, "dy": 2.0 * (y - t.double()) / t.numel(), "gradients": p.grad}
