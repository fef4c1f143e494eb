"""Timed workloads of the framework through its public entry points (Context.trace,
Context.chem_step, Context.rt_timestep, MLP.train), from single-source calls bound by latency
to the largest lognormal configuration.

A case is a dict of plain values. Its "kind" says what one pass does:

  trace     one radiation field: rays from every source, rates out
  step      a whole RT step as a run makes it: trace, time-step limits, chemistry (in place)
  chem      the plain chemistry step (in place)
  learned   the gated learned chemistry step with the plain fallback (in place)
  timestep  the two limits of the adaptive time step
  train     training of the learned step's network from samples

Inputs are drawn on the GPU from the seed alone. exact() holds the same mathematics in 64-bit
torch operations.
"""
import math

import numpy as np
import torch

from paper_1807_07094_amd import arc
from paper_1807_07094_amd import workload as W

DEV = "cuda"
TAU_THIN = float(np.float32(0.1))
NET_PARAMS = 8 * 64 + 64 + 64 * 64 + 64 + 64 * 2 + 2  # weights and biases of the 8-64-64-2 network
EDGES = {2: (13.6, 24.6), 3: (13.6, 24.6, 54.4), 4: (13.6, 24.6, 39.0, 54.4)}

TRACE = {"kind": "trace", "bins": 3, "level0": 1, "eps": 1e-6, "field": "lognormal", "place": "top1",
         "correction": "none", "precision": "fp32_comp", "thin": False, "graph": False}
GAS = {"helium": True, "dt_myr": 0.1}


def listed():
    return [
        # the smallest call: a ragged grid and three sources, a handful of short launches
        dict(TRACE, name="trace-28x32x24-3src", nx=28, ny=32, nz=24, nsrc=3, place="uniform"),
        # the HII-region test's time loop: one source in hydrogen, a whole step per pass
        dict(TRACE, name="step-64-1src", kind="step", nx=64, ny=64, nz=64, nsrc=1, bins=1, level0=0, eps=1e-12,
             field="uniform", place="centre", graph=True, dt_myr=0.02),
        # the cosmic density-field test: few sources, one per many cells
        dict(TRACE, name="trace-128-16src", nx=128, ny=128, nz=128, nsrc=16, place="uniform", graph=True),
        # many sources in a mid-size box, the ordinary production shape
        dict(TRACE, name="trace-256-1024src", nx=256, ny=256, nz=256, nsrc=1024),
        # the largest: thousands of sources, recorded launches as a long run replays them
        dict(TRACE, name="trace-512-4096src", nx=512, ny=512, nz=512, nsrc=4096, graph=True),
        # a slab whose sides are no multiples of the layout's blocks, two bands, smooth density
        dict(TRACE, name="trace-203x100x37-200src", nx=203, ny=100, nz=37, nsrc=200, bins=2, field="smooth"),
        # the photon-conserving geometric correction
        dict(TRACE, name="trace-corr-192-128src", nx=192, ny=192, nz=192, nsrc=128, correction="conserving"),
        # ionised bubbles around the sources, thin spheres in and measured radii out
        dict(TRACE, name="trace-thin-128-32src", nx=128, ny=128, nz=128, nsrc=32, place="uniform", thin=True),
        # chemistry of hydrogen and helium gas with fronts, bubbles and neutral cells
        dict(GAS, name="chem-256", kind="chem", nx=256, ny=256, nz=256),
        # the same gas through the learned step and its gate
        dict(GAS, name="learned-256", kind="learned", nx=256, ny=256, nz=256, graph=True, samples=131072),
        # the limits that choose the next step
        dict(GAS, name="timestep-320", kind="timestep", nx=320, ny=320, nz=320),
        # training of the network on sampled states
        {"name": "train-65536", "kind": "train", "samples": 65536, "batch": 1024, "epochs": 4},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["trace"] * 6 + ["step", "chem", "chem", "learned", "timestep", "train"])
    if kind == "train":
        return {"kind": "train", "samples": log_int(8000, 131072), "batch": rng.choice([256, 1000, 1024, 2048]),
                "epochs": rng.randint(1, 4)}
    if kind in ("trace", "step"):
        n = log_int(20, 288)
        dims = [max(9, min(320, int(n * rng.uniform(0.6, 1.5)))) for _ in range(3)]
        corr = rng.choice(["none", "none", "none", "conserving", "conserving", "fc", "fc_squared"])
        thin = corr == "none" and rng.random() < 0.2
        case = dict(TRACE, kind=kind, nx=dims[0], ny=dims[1], nz=dims[2], nsrc=log_int(1, 24 if thin else 300),
                    bins=rng.choice([1, 2, 3, 3, 3, 4]), level0=rng.choice([0, 1, 1, 1]),
                    eps=rng.choice([1e-6, 1e-6, 1e-12]), field=rng.choice(["lognormal", "smooth", "uniform"]),
                    place=rng.choice(["uniform", "top1"]), correction=corr, thin=thin, graph=rng.random() < 0.5)
        if corr == "none" and not thin and rng.random() < 0.15:
            case["precision"] = "fp32_plain"
        if kind == "step":
            case.update(thin=False, precision="fp32_comp", dt_myr=rng.choice([0.02, 0.05]))
        return case
    n = log_int(24, 288)
    case = dict(GAS, kind=kind, **{k: max(9, int(n * rng.uniform(0.7, 1.3))) for k in ("nx", "ny", "nz")},
                dt_myr=rng.choice([0.02, 0.1, 0.5]))
    if kind == "learned":
        case.update(graph=rng.random() < 0.5, samples=log_int(30000, 131072))
    else:
        case["helium"] = rng.random() < 0.75
    return case


# ----------------------------------------------------------------------------------
# Inputs.
# ----------------------------------------------------------------------------------
def _bins(nb):
    return W.bins_monochromatic(13.6) if nb == 1 else W.bins_blackbody(1e5, EDGES[nb])


def _density(case, gen):
    shape = (case["nz"], case["ny"], case["nx"])
    field = case.get("field", "lognormal")
    if field == "uniform":
        return torch.full(shape, 1e-3, device=DEV)
    g = torch.randn(shape, generator=gen, device=DEV)
    if field == "lognormal":
        return (1e-3 * torch.exp(g - 0.5)).contiguous()
    gk = torch.fft.rfftn(g)
    for axis in range(3):  # periodic Gaussian smoothing over two cells
        k = (torch.fft.rfftfreq if axis == 2 else torch.fft.fftfreq)(shape[axis], device=DEV)
        view = [1, 1, 1]
        view[axis] = -1
        gk *= torch.exp(-0.5 * (2 * math.pi * k * 2.0) ** 2).view(view)
    g = torch.fft.irfftn(gk, s=shape)
    g = (g - g.mean()) / g.std()
    return (1e-3 * torch.exp(0.5 * g - 0.125)).contiguous()


def _neutral(n_h, helium):
    full = torch.full_like
    return {"n_h": n_h, "x_hi": full(n_h, 1.0 - 1.2e-3), "x_hei": full(n_h, 1.0 - 1.2e-3 if helium else 0.0),
            "x_heii": full(n_h, 1.2e-3 if helium else 0.0), "temp": full(n_h, 1e4),
            "cell_cm": W.COSMIC_CELL_CM, "y_he": 0.08 if helium else 0.0}


def _distance2(shape, pos):
    nz, ny, nx = shape
    x, y, z = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5 for n in (nx, ny, nz))
    return ((z - pos[2]) ** 2).view(-1, 1, 1) + ((y - pos[1]) ** 2).view(1, -1, 1) + ((x - pos[0]) ** 2).view(1, 1, -1)


def _trace_inputs(case, seed):
    """Grid, sources and bins of a trace: power-law luminosities, sources on the 2^-12 lattice."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    n_h = _density(case, gen)
    ns, nb = case["nsrc"], case["bins"]
    grid = _neutral(n_h, nb > 1)
    nz, ny, nx = n_h.shape
    if case["place"] == "centre":
        pos = np.array([[nx / 2, ny / 2, nz / 2]])
        ndot = np.array([5e48 * (1.0 + 0.1 * rng.random())])
        grid["cell_cm"] = 6.6 * W.KPC_CM / nx
    else:
        if case["place"] == "top1" and case["field"] != "uniform":
            cand = torch.topk(n_h.view(-1), max(ns, n_h.numel() // 100)).indices.cpu().numpy()
            cells = np.sort(rng.choice(np.sort(cand), ns, replace=False))
        else:
            cells = np.sort(rng.choice(n_h.numel(), ns, replace=False))
        z, rem = np.divmod(cells, ny * nx)
        y, x = np.divmod(rem, nx)
        pos = np.stack([x, y, z], 1) + rng.integers(0, W.LATTICE, (ns, 3)) / W.LATTICE
        u = rng.random(ns)
        ndot = 1.0 / (1e-48 - u * (1e-48 - 1e-51))
    src = {"pos": np.ascontiguousarray(pos, np.float64), "ndot": np.ascontiguousarray(ndot, np.float64)}
    if case["thin"]:
        # bubbles of an evolved run: radius with the cube root of the luminosity, the last
        # trace's thin radius somewhat inside
        rad = np.clip(9.0 * (ndot / 1e49) ** (1.0 / 3.0), 3.0, 26.0) * rng.uniform(0.85, 1.15, ns)
        for p, r in zip(pos, rad):
            inside = _distance2(n_h.shape, p) < r * r
            grid["x_hi"][inside] = 2e-4
            grid["temp"][inside] = 1.6e4
            if nb > 1:
                grid["x_hei"][inside] = 3e-4
                grid["x_heii"][inside] = 0.6
        src["r_thin"] = np.maximum(0.0, rad - rng.uniform(0.5, 2.0, ns))
        src["r_thin_out"] = np.zeros(ns)
    return grid, src, _bins(nb)


def _gas_inputs(case, seed):
    """A grid inside a run: bubbles around a few sources, with the rates they cause, gas that has
    relaxed towards them for 10 Myr, and temperatures of photoheated gas."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    n_h = _density(case, gen)
    helium = case["helium"]
    grid = _neutral(n_h, helium)
    bins = _bins(3 if helium else 1)
    L, sig = grid["cell_cm"], bins["sigma"]
    shape = n_h.shape
    excess = np.maximum(bins["e_erg"][:, None] - bins["e_thr"][None, :], 0.0)
    gamma = torch.zeros((3,) + tuple(shape), device=DEV)
    heat = torch.zeros_like(gamma)
    kap = 1e-3 * L * (sig[:, 0] + grid["y_he"] * sig[:, 1])
    size = min(shape)
    for _ in range(12):
        pos = rng.random(3) * np.array(shape[::-1])
        rad = size * rng.uniform(0.06, 0.22)
        ndot = 2.0e50 * (rad / 25.0) ** 3
        r2 = _distance2(shape, pos)
        deep = torch.clamp(r2.sqrt() - rad, min=0.0)
        inv = 1.0 / (4 * math.pi * torch.clamp(r2, min=0.25) * L * L)
        for b, f in enumerate(bins["frac"]):
            flux = ndot * f * torch.exp(-kap[b] * deep) * inv
            for s in range(3):
                if sig[b, s] > 0:
                    gamma[s] += (flux * sig[b, s]).float()
                    heat[s] += (flux * (sig[b, s] * excess[b, s])).float()
    age = 10.0 * W.MYR_S
    x_eq = 2.6e-13 * n_h / (2.6e-13 * n_h + gamma[0])
    x = x_eq + (1.0 - 1.2e-3 - x_eq) * torch.exp(-gamma[0] * age)
    grid["x_hi"] = torch.clamp(x, 1e-7, 1.0 - 1.2e-3)
    if helium:
        e1, e2 = 4e-13 * n_h / (4e-13 * n_h + gamma[1]), 2e-12 * n_h / (2e-12 * n_h + gamma[2])
        x1 = e1 + (1.0 - 1.2e-3 - e1) * torch.exp(-gamma[1] * age)
        x2 = (1.0 - x1) * (e2 + (1.0 - e2) * torch.exp(-gamma[2] * age))
        grid["x_hei"], grid["x_heii"] = torch.clamp(x1, 0.0, 1.0 - 1.2e-3), torch.clamp(x2, 0.0, 1.0)
    noise = torch.rand(shape, generator=gen, device=DEV)
    grid["temp"] = (1e4 * (0.7 + 0.6 * noise) * (1.0 + 0.9 * (1.0 - grid["x_hi"]))).contiguous()
    chem = {"isothermal": 0, "rates": 1, "collisional": 1, "alpha_hii": 2.59e-13, "eps": 0.1, "max_sub": 100000,
            "t_floor": 1.0} if helium else _test1_chem()
    return grid, gamma, heat, bins, chem


def _test1_chem():
    return {"isothermal": 1, "rates": 0, "collisional": 0, "alpha_hii": 2.59e-13, "eps": 0.1, "max_sub": 100000,
            "t_floor": 1.0}


def _samples(m, seed):
    """Training samples: cells of such a grid, 32 log-spaced time steps, 64-bit targets."""
    grid, gamma, heat, _, chem = _gas_inputs({"nx": 96, "ny": 96, "nz": 96, "helium": True, "field": "lognormal"}, seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) + 7)
    pick = torch.randint(0, grid["n_h"].numel(), (m,), generator=gen, device=DEV)
    flat = {k: grid[k].reshape(-1)[pick] for k in ("n_h", "x_hi", "x_hei", "x_heii", "temp")}
    flat.update(cell_cm=grid["cell_cm"], y_he=grid["y_he"])
    ga, he = gamma.reshape(3, -1)[:, pick], heat.reshape(3, -1)[:, pick]
    steps = torch.logspace(-3, 0, 32, dtype=torch.float64, device=DEV) * W.MYR_S
    dt = steps[torch.randint(0, 32, (m,), generator=gen, device=DEV)]
    out = _exact_chem(flat, ga, he, dt, chem)
    h = he[0] * flat["x_hi"] + grid["y_he"] * (he[1] * flat["x_hei"] + he[2] * flat["x_heii"])
    X = torch.stack([flat["n_h"], flat["x_hi"], flat["temp"], ga[0], dt.float(), h, flat["x_heii"], flat["x_hei"]], 1)
    Y = torch.stack([out["x_hi"], out["temp"]], 1).float()
    return X.contiguous(), Y.contiguous()


# ----------------------------------------------------------------------------------
# Preparation, one pass, and the work it cannot do without.
# ----------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case, "ctx": arc.Context(0)}
    if kind == "train":
        state["X"], state["Y"] = _samples(case["samples"], seed)
        state["net"] = arc.MLP(state["ctx"])
        return state
    if kind in ("trace", "step"):
        state["grid"], state["src"], state["bins"] = _trace_inputs(case, seed)
        shape = (3,) + tuple(state["grid"]["n_h"].shape)
        state["gamma"] = torch.empty(shape, device=DEV)
        state["heat"] = torch.empty(shape, device=DEV)
        helium = case["bins"] > 1
        state["chem"] = {"isothermal": 0, "rates": 1, "collisional": 1, "alpha_hii": 2.59e-13, "eps": 0.1,
                         "max_sub": 100000, "t_floor": 1.0} if helium else _test1_chem()
    else:
        state["grid"], state["gamma"], state["heat"], state["bins"], state["chem"] = _gas_inputs(case, seed)
        if kind == "learned":
            X, Y = _samples(case["samples"], 5)
            state["net"] = arc.MLP(state["ctx"])
            state["net"].train(X, Y, epochs=6, batch=1024, lr=2e-3, seed=3, y_he=0.08)
    return state


def _gas_out(grid):
    return {k: grid[k] for k in ("x_hi", "x_hei", "x_heii", "temp")}


def run(state):
    case, ctx, kind = state["case"], state["ctx"], state["case"]["kind"]
    if kind == "train":
        net = state["net"]
        rep = net.train(state["X"], state["Y"], epochs=case["epochs"], batch=case["batch"], lr=2e-3, seed=3)
        weights = np.frombuffer(net.save()[-4 * NET_PARAMS:], np.float32)
        return {"weights": weights, "val_rmse_x": rep["val_rmse_x"], "val_rmse_logt": rep["val_rmse_logt"]}
    grid, gamma, heat = state["grid"], state["gamma"], state["heat"]
    out = {}
    if kind in ("trace", "step"):
        led = ctx.trace(grid, state["src"], state["bins"], W.MYR_S, gamma, heat, level0=case["level0"],
                        eps_term=case["eps"], precision=case["precision"], graph=case["graph"],
                        correction=case["correction"])
        out = {"gamma": gamma, "heat": heat, "absorbed": led["absorbed"], "escaped": led["escaped"],
               "crossings": led["crossings"], "rays": led["rays"]}
        if case["thin"]:
            out["r_thin"] = state["src"]["r_thin_out"]
    if kind in ("timestep", "step"):
        c = state["chem"]
        out["dt"] = ctx.rt_timestep(grid, gamma, state["bins"], rates=c["rates"], collisional=c["collisional"],
                                    alpha_hii=c["alpha_hii"])
    if kind in ("chem", "learned", "step"):
        more = {"mode": "mlp_gated", "mlp": state["net"]} if kind == "learned" else {}
        ctx.chem_step(grid, gamma, heat, case["dt_myr"] * W.MYR_S, graph=case.get("graph", False), **state["chem"],
                      **more)
        out.update(_gas_out(grid))
    return out


def _crossings(case):
    """About how many (ray, cell) segments a trace makes: 3/2 per cell of path length, and at
    radius r the rays of the first level whose split radius lies beyond r, out to the radius
    where the hardest band is attenuated or the box ends."""
    b = _bins(case["bins"])
    neutral = 1e-3 * (6.6 * W.KPC_CM / case["nx"] if case["place"] == "centre" else W.COSMIC_CELL_CM)
    kap = min(neutral * (s[0] + (0.08 * (s[1] + 1e-3 * s[2]) if case["bins"] > 1 else 0.0)) for s in b["sigma"])
    side = (case["nx"] * case["ny"] * case["nz"]) ** (1.0 / 3.0)
    end = min(-math.log(case["eps"]) / kap + (9.0 if case["thin"] else 0.0), 0.55 * side)
    base, level, r, total = math.sqrt(3.0 / (4.0 * math.pi)), case["level0"], 0.0, 0.0
    while r < end:
        nxt = min(end, base * 2.0 ** level)
        total += 12.0 * 4.0 ** level * 1.5 * max(0.0, nxt - r)
        r, level = max(r, nxt), level + 1
    return case["nsrc"] * total


def work(case):
    kind = case["kind"]
    if kind == "train":
        m = case["samples"] * case["epochs"]
        return {"bytes": 40.0 * m, "flops": 6.0 * NET_PARAMS * m}
    cells = case["nx"] * case["ny"] * case["nz"]
    bytes_, flops = 0.0, 0.0
    if kind in ("trace", "step"):
        states = 4 if case["bins"] > 1 else 2
        bytes_ += (4.0 * states + 24.0) * cells + 32.0 * case["nsrc"]
        flops += _crossings(case) * (25.0 + 15.0 * case["bins"])
    if kind in ("timestep", "step"):
        bytes_ += 24.0 * cells
        flops += 80.0 * cells
    if kind in ("chem", "learned", "step"):
        bytes_ += 60.0 * cells
        flops += (300.0 if kind != "learned" else 300.0 + 2.0 * NET_PARAMS) * cells
    return {"bytes": float(bytes_), "flops": float(flops)}


# ----------------------------------------------------------------------------------
# The same in 64 bits.
# ----------------------------------------------------------------------------------
def _pixel_dirs(level, pix):
    """HEALPix centres, nested order, rounded to float32 as the method takes them."""
    ns = 1 << level
    face, q = pix // (ns * ns), pix % (ns * ns)
    x, y = torch.zeros_like(q), torch.zeros_like(q)
    for b in range(level):
        x |= ((q >> (2 * b)) & 1) << b
        y |= ((q >> (2 * b + 1)) & 1) << b
    row, col = face // 4, face % 4
    ring = (row + 2) * ns - x - y - 1
    north, south = ring < ns, ring > 3 * ns
    nr = torch.where(north, ring, torch.where(south, 4 * ns - ring, torch.full_like(ring, ns)))
    cap = (north | south)
    shift = torch.where(cap, torch.zeros_like(ring), (ring - ns) & 1)
    polar = 1.0 - nr.double() ** 2 / (3.0 * ns * ns)
    z = torch.where(north, polar, torch.where(south, -polar, 2.0 * (2 * ns - ring).double() / (3.0 * ns)))
    lon = 2 * col + torch.where(row == 1, torch.zeros_like(row), torch.ones_like(row))
    j = (lon * nr + x - y + 1 + shift) // 2
    j = torch.where(j > 4 * nr, j - 4 * nr, torch.where(j < 1, j + 4 * nr, j))
    # phi as whole quarter turns and the rest, so that directions along an axis are exactly so
    num, den = 2 * j - 1 - shift, 2 * nr
    quarter, rest = num // den, 0.5 * math.pi * (num % den).double() / den.double()
    ca, sa = torch.cos(rest), torch.sin(rest)
    cx = torch.where(quarter == 0, ca, torch.where(quarter == 1, -sa, torch.where(quarter == 2, -ca, sa)))
    cy = torch.where(quarter == 0, sa, torch.where(quarter == 1, ca, torch.where(quarter == 2, -sa, -ca)))
    st = torch.sqrt((1.0 - z) * (1.0 + z))
    return torch.stack([st * cx, st * cy, z], 1).float().double()


def _exact_trace(case, grid, src, bins):
    n_h = grid["n_h"].double().reshape(-1)
    shape = grid["n_h"].shape
    dims = torch.tensor([shape[2], shape[1], shape[0]], device=DEV)
    stride = torch.tensor([1, shape[2], shape[2] * shape[1]], device=DEV)
    L, y, nb = grid["cell_cm"], grid["y_he"], case["bins"]
    sig = bins["sigma"]
    xs3 = [grid[k].double().reshape(-1) for k in ("x_hi", "x_hei", "x_heii")]
    kappa = torch.stack([L * n_h * (sig[b, 0] * xs3[0] + y * (sig[b, 1] * xs3[1] + sig[b, 2] * xs3[2]))
                         for b in range(nb)], 1)
    J = torch.zeros((n_h.numel(), nb), dtype=torch.float64, device=DEV)
    escaped = torch.zeros((), dtype=torch.float64, device=DEV)
    pos = torch.from_numpy(src["pos"]).to(DEV)
    rate = torch.from_numpy(src["ndot"][:, None] * bins["frac"][None, :]).to(DEV)
    base = np.float32(math.sqrt(3.0 / (4.0 * math.pi)))
    diag = math.sqrt(sum(float(v) ** 2 for v in shape))
    lmax = 0
    while float(base) * 2.0 ** lmax < diag:
        lmax += 1

    def split_radius(level):
        return float(base) * 2.0 ** level if level < lmax else math.inf

    tau_end = float(np.float32(-math.log(case["eps"])))
    soft, thin, corr = int(np.argmin(bins["e_erg"])), case["thin"], case["correction"]
    r_min = torch.full((len(src["ndot"]),), math.inf, dtype=torch.float64, device=DEV)
    r_thin = torch.zeros(len(src["ndot"]), dtype=torch.float64, device=DEV)
    if thin:
        r_thin = torch.from_numpy(src["r_thin"].astype(np.float32).astype(np.float64)).to(DEV)
        for s in range(len(src["ndot"])):
            d2 = _distance2(shape, src["pos"][s]).reshape(-1)
            cells = torch.nonzero(d2 < r_thin[s] ** 2).flatten()
            J[cells] += rate[s][None, :] / (4 * math.pi * torch.clamp(d2[cells], min=0.25))[:, None]
    ns, npix = len(src["ndot"]), 12 * 4 ** case["level0"]
    every = torch.arange(ns * npix, device=DEV)
    stack = [(case["level0"], every // npix, every % npix, torch.zeros((ns * npix, nb), dtype=torch.float64, device=DEV))]
    piece = 3_000_000
    while stack:
        level, s, pix, tau = stack.pop()
        if s.numel() > piece:
            stack.append((level, s[piece:], pix[piece:], tau[piece:]))
            s, pix, tau = s[:piece], pix[:piece], tau[:piece]
        d, xs = _pixel_dirs(level, pix), pos[s]
        w = rate[s] / (12.0 * 4.0 ** level)
        t = torch.full((s.numel(),), 0.0 if level == case["level0"] else split_radius(level - 1), dtype=torch.float64,
                       device=DEV)
        if thin:
            t = torch.maximum(t, r_thin[s])
        t_end = split_radius(level)
        done = [[], [], []]
        once = t >= t_end  # inside the thin sphere: split without a crossing
        if thin and bool(once.any()):
            done = [[s[once]], [pix[once]], [tau[once]]]
        e = d.abs()
        p = xs + t[:, None] * d
        c = torch.floor(p)
        c = torch.where((d < 0) & (c == p), c - 1, c).long()
        step = torch.sign(d).long()
        inside = ((c >= 0) & (c < dims)).all(1)
        gone = ~inside & ~once
        if bool(gone.any()):
            escaped += (w[gone] * torch.exp(-tau[gone])).sum()
            if thin:
                early = gone & (tau[:, soft] < TAU_THIN)
                r_min.scatter_reduce_(0, s[early], t[early], "amin")
        keep = torch.nonzero(inside & ~once).flatten()
        s, pix, tau, d, e, xs, w, t, c, step = (v[keep] for v in (s, pix, tau, d, e, xs, w, t, c, step))
        lpix = math.sqrt(math.pi / 3.0) * 2.0 ** -level
        while s.numel():
            a = torch.where(step < 0, xs - c, c + 1 - xs)
            ti = torch.where(e > 0, a / e, torch.full_like(a, math.inf))
            tb = ti.min(1).values
            at_end = tb >= t_end
            tn = torch.clamp(tb, max=t_end)
            ds = torch.clamp(tn - t, min=0.0)
            cell = (c * stride).sum(1)
            k = kappa[cell]
            dtau = k * ds[:, None]
            through = torch.exp(-tau)
            v = torch.where(k > 0, w * through * -torch.expm1(-dtau) / torch.where(k > 0, k, torch.ones_like(k)),
                            w * through * ds[:, None])
            if thin:
                ts, dts = tau[:, soft], dtau[:, soft]
                hit = (ts < TAU_THIN) & (ts + dts >= TAU_THIN)
                r_min.scatter_reduce_(0, s[hit], (t + (TAU_THIN - ts) / k[:, soft])[hit], "amin")
            tau = tau + dtau
            after = w * torch.exp(-tau)
            ended = ((tau >= tau_end) & (dtau >= 0.01)).all(1)
            v = torch.where(ended[:, None], v + after / torch.where(k > 0, k, torch.ones_like(k)), v)
            if corr != "none":
                tm = 0.5 * (t + tn)
                ahead = a - tm[:, None] * e
                up = step >= 0
                hi, lo = torch.where(up, ahead, 1.0 - ahead), torch.where(up, 1.0 - ahead, ahead)
                upper = hi < lo - 1e-9
                di = torch.where(upper, hi, lo)
                dmin, axis = torch.full_like(tm, math.inf), torch.zeros_like(cell)
                side = -torch.ones_like(cell)
                for i in range(3):
                    better = di[:, i] < dmin - 1e-9
                    dmin = torch.where(better, di[:, i], dmin)
                    axis = torch.where(better, torch.full_like(axis, i), axis)
                    side = torch.where(better, torch.where(upper[:, i], 1, -1), side)
                fc = torch.where(dmin < 0.5 * lpix * tm, 0.5 + dmin / (lpix * tm), torch.ones_like(dmin))
                if corr == "fc_squared":
                    fc = fc * fc
                if corr == "conserving":
                    ca = c.gather(1, axis[:, None])[:, 0] + side
                    ok = (fc < 1) & (ca >= 0) & (ca < dims[axis])
                    other = torch.where(ok, cell + side * stride[axis], cell)
                    kn = kappa[other]
                    move = ok[:, None] & (kn > 0)
                    moved = torch.where(move, (1.0 - fc)[:, None] * v, torch.zeros_like(v))
                    J.index_add_(0, other, moved * k / torch.where(kn > 0, kn, torch.ones_like(kn)))
                    v = v - moved
                else:
                    v = v * fc[:, None]
            J.index_add_(0, cell, v)
            c = c + step * ((ti <= tn[:, None]) & ~at_end[:, None])
            t = tn
            inside = ((c >= 0) & (c < dims)).all(1)
            out = ~inside & ~ended & ~at_end
            escaped += after[out].sum()
            if thin:
                early = out & (tau[:, soft] < TAU_THIN)
                r_min.scatter_reduce_(0, s[early], t[early], "amin")
            sp = torch.nonzero(at_end & ~ended).flatten()
            for to, what in zip(done, (s, pix, tau)):
                to.append(what[sp])
            keep = torch.nonzero(inside & ~ended & ~at_end).flatten()
            s, pix, tau, d, e, xs, w, t, c, step = (q[keep] for q in (s, pix, tau, d, e, xs, w, t, c, step))
        if done[0]:
            s, pix, tau = (torch.cat(v) for v in done)
            if s.numel():
                child = (4 * pix[:, None] + torch.arange(4, device=DEV)).reshape(-1)
                stack.append((level + 1, s.repeat_interleave(4), child, tau.repeat_interleave(4, 0)))
    excess = np.maximum(bins["e_erg"][:, None] - bins["e_thr"][None, :], 0.0)
    ga = J @ torch.from_numpy(sig / L ** 2).to(DEV)
    he = J @ torch.from_numpy(sig * excess / L ** 2).to(DEV)
    out = {"gamma": ga.T.reshape((3,) + tuple(shape)), "heat": he.T.reshape((3,) + tuple(shape)),
           "absorbed": float((J * kappa).sum()) * W.MYR_S, "escaped": float(escaped) * W.MYR_S,
           "crossings": None, "rays": None}
    if thin:
        out["r_thin"] = r_min.cpu().numpy()
    return out


T_HI, T_HEI, T_HEII, K_B, EV = 157807.0, 285335.0, 631515.0, 1.380649e-16, 1.602176634e-12


def _coefficients(T):
    """Hui & Gnedin (1997) case-B fits, lambda = 2 T_i / T."""
    l1, l2, l3 = 2 * T_HI / T, 2 * T_HEI / T, 2 * T_HEII / T
    diel = 1.90e-3 * T ** -1.5 * torch.exp(-0.375 * l3) * (1 + 0.3 * torch.exp(-0.075 * l3))
    return {"hii": 2.753e-14 * l1 ** 1.5 / (1 + (l1 / 2.740) ** 0.407) ** 2.242, "heii": 1.26e-14 * l2 ** 0.75 + diel,
            "heiii": 2 * 2.753e-14 * l3 ** 1.5 / (1 + (l3 / 2.740) ** 0.407) ** 2.242,
            "khi": 21.11 * T ** -1.5 * torch.exp(-l1 / 2) * l1 ** -1.089 / (1 + (l1 / 0.354) ** 0.874) ** 1.101,
            "khei": 32.38 * T ** -1.5 * torch.exp(-l2 / 2) * l2 ** -1.146 / (1 + (l2 / 0.416) ** 0.987) ** 1.056,
            "kheii": 19.95 * T ** -1.5 * torch.exp(-l3 / 2) * l3 ** -1.089 / (1 + (l3 / 0.553) ** 0.735) ** 1.275,
            "diel": diel, "l1": l1, "l2": l2, "l3": l3}


def _cooling(T, k, ne, nhi, nhii, nhei, nheii, nheiii):
    l1, l2, l3 = k["l1"], k["l2"], k["l3"]
    rec1 = 3.435e-30 * T * l1 ** 1.970 / (1 + (l1 / 2.250) ** 0.376) ** 3.720
    rec3 = 2 * 3.435e-30 * T * l3 ** 1.970 / (1 + (l3 / 2.250) ** 0.376) ** 3.720
    rec2 = K_B * T * 1.26e-14 * l2 ** 0.75 + 0.75 * 54.418 * EV * k["diel"]
    damp = 1.0 / (1.0 + torch.sqrt(T / 1e5))
    gff = 1.1 + 0.34 * torch.exp(-(5.5 - torch.log10(T)) ** 2 / 3.0)
    return ne * (rec1 * nhii + rec2 * nheii + rec3 * nheiii + EV * (13.598 * k["khi"] * nhi + 24.587 * k["khei"] * nhei +
                                                                    54.418 * k["kheii"] * nheii)
                 + 7.5e-19 * torch.exp(-0.375 * l1) * damp * nhi
                 + 5.54e-17 * T ** -0.397 * torch.exp(-0.375 * l3) * damp * nheii
                 + 1.42e-27 * gff * torch.sqrt(T) * (nhii + nheii + 4 * nheiii))


def _exact_chem(grid, gamma, heat, dt, chem):
    """Backward difference, sub-cycled: each sub-step at most eps of the shortest change time.
    dt: seconds, a number or one per cell."""
    shape, y = grid["n_h"].shape, grid["y_he"]
    f = {k: grid[k].double().reshape(-1) for k in ("n_h", "x_hi", "x_hei", "x_heii", "temp")}
    ga, he = gamma.double().reshape(3, -1), heat.double().reshape(3, -1)
    nh = f["n_h"]
    end = dt if torch.is_tensor(dt) else torch.full_like(nh, dt)
    S = [nh, nh * f["x_hi"], y * nh * f["x_hei"], torch.clamp(y * nh * (1 - f["x_hei"] - f["x_heii"]), min=0.0),
         y * nh * f["x_heii"], f["temp"], torch.zeros_like(nh), end, ga[0], ga[1], ga[2], he[0], he[1], he[2]]
    nhii, ne = nh - S[1], nh - S[1] + S[4] + 2 * S[3]
    S += [ne, 1.5 * K_B * S[5] * (nh + y * nh + ne)]
    res = {k: torch.empty_like(nh) for k in ("x_hi", "x_hei", "x_heii", "temp")}
    idx = torch.arange(nh.numel(), device=nh.device)
    eps, inf = chem["eps"], math.inf
    while idx.numel():
        nh, nhi, nhei, nheiii, nheii, T, t, end, g0, g1, g2, h0, h1, h2, ne, E = S
        nhe, nhii = y * nh, nh - nhi
        if chem["rates"]:
            k = _coefficients(T)
        else:
            zero = torch.zeros_like(T)
            k = {"hii": zero + chem["alpha_hii"], "heii": zero, "heiii": zero, "khi": zero, "khei": zero, "kheii": zero}
        dn = k["hii"] * ne * nhii - (g0 + k["khi"] * ne) * nhi
        edot = torch.zeros_like(T)
        if not chem["isothermal"]:
            edot = nhi * h0 + nhei * h1 + nheii * h2 - _cooling(T, k, ne, nhi, nhii, nhei, nheii, nheiii)
        lim = torch.full_like(T, inf)
        lim = torch.where(edot != 0, eps * E / edot.abs(), lim)
        lim = torch.where((nhi > 0) & (dn != 0), torch.minimum(lim, eps * nhi / dn.abs()), lim)
        lim = torch.where((nhii > 0) & (dn != 0), torch.minimum(lim, eps * nhii / dn.abs()), lim)
        last = ~(lim < end - t)
        h = torch.minimum(lim, end - t)
        nhi = torch.minimum((nhi + k["hii"] * ne * nhii * h) / (1 + (g0 + k["khi"] * ne) * h), nh)
        a = (nhei + k["heii"] * ne * nheii * h) / (1 + (g1 + k["khei"] * ne) * h)
        b = (nheiii + (g2 + k["kheii"] * ne) * nheii * h) / (1 + k["heiii"] * ne * h)
        nhei = torch.minimum(a, nhe)
        nheiii = torch.minimum(b, nhe - nhei)
        nheii = torch.clamp(nhe - nhei - nheiii, min=0.0)
        ne = nh - nhi + nheii + 2 * nheiii
        if not chem["isothermal"]:
            part = 1.5 * K_B * (nh + nhe + ne)
            T = torch.clamp((E + edot * h) / part, min=chem["t_floor"])
            E = torch.maximum(E + edot * h, chem["t_floor"] * part)
        fin = idx[last]
        res["x_hi"][fin] = (nhi / nh)[last]
        if y > 0:
            res["x_hei"][fin], res["x_heii"][fin] = (nhei / nhe)[last], (nheii / nhe)[last]
        else:
            res["x_hei"][fin], res["x_heii"][fin] = f["x_hei"][fin], f["x_heii"][fin]
        res["temp"][fin] = T[last]
        keep = torch.nonzero(~last).flatten()
        idx = idx[keep]
        S = [v[keep] for v in (nh, nhi, nhei, nheiii, nheii, T, t + h, end, g0, g1, g2, h0, h1, h2, ne, E)]
    return {k: v.reshape(shape) for k, v in res.items()}


def _exact_timestep(grid, gamma, bins, chem):
    nh = grid["n_h"].double()
    nhi, nhe = nh * grid["x_hi"], grid["y_he"] * nh
    nheii = nhe * grid["x_heii"]
    ne = nh - nhi + nheii + 2 * torch.clamp(nhe - nhe * grid["x_hei"] - nheii, min=0.0)
    if chem["rates"]:
        k = _coefficients(grid["temp"].double())
        a, kh = k["hii"], k["khi"] * (1.0 if chem["collisional"] else 0.0)
    else:
        a, kh = chem["alpha_hii"], 0.0
    dn = (a * ne * (nh - nhi) - (gamma[0].double() + kh * ne) * nhi).abs()
    sl = float(bins["sigma"][0, 0]) * grid["cell_cm"]
    thick = (nhi * sl > 0.5) & (dn > 0)
    one = torch.where(thick, 0.1 * nhi / dn, torch.full_like(dn, math.inf)).min()
    two = torch.where(dn > 0, 0.1 / (sl * dn), torch.full_like(dn, math.inf)).min()
    return float(one), float(two)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("train", "learned"):  # the network's arithmetic is 16-bit by design
        return None
    if kind in ("trace", "step"):
        if _crossings(case) > 6e9:  # longer than it is worth
            return None
        grid, src, bins = _trace_inputs(case, seed)
        out = _exact_trace(case, grid, src, bins)
        gamma, heat = out["gamma"], out["heat"]
        helium = case["bins"] > 1
        chem = {"isothermal": 0, "rates": 1, "collisional": 1, "alpha_hii": 2.59e-13, "eps": 0.1,
                "t_floor": 1.0} if helium else _test1_chem()
    else:
        grid, gamma, heat, bins, chem = _gas_inputs(case, seed)
        out = {}
    if kind in ("timestep", "step"):
        out["dt"] = _exact_timestep(grid, gamma, bins, chem)
    if kind in ("chem", "step"):
        out.update(_exact_chem(grid, gamma, heat, case["dt_myr"] * W.MYR_S, chem))
    return out
