"""Timed cases of the ray-tracing library, through its public entry points.

`listed()` names the workloads, `draw(rng)` gives more of the same ranges,
`prepare(case, seed)` makes what a program holds before the call (fields,
sources, context, outputs), `run(state)` is one pass, `work(case)` the bytes
and operations the pass cannot do without and `exact(case, seed)` the same
outputs in plain float64 torch, from the method's formulas alone.

A case is a dict of plain values:
  path     forward   Gamma of a source list
           column    Gamma and the entry column of one source
           static    Gamma through the entry point that allocates nothing
           heating   Gamma and the photo-heating rate
           helium    Gamma of HI and of HeI (four bands)
           fwd_adj   Gamma, then the adjoint with the columns recomputed
           step      the differentiable forward (records kept) and its backward
           chemistry one chemistry pass of the time step
  N, cell  grid side and cell size (cm)
  n_src, R_lo, R_hi, lgQ_lo, lgQ_hi   sources: radii (cells) and log10 of the photon rates
  field    uniform, bubbles (n_bub ionized balls, around the sources first) or
           smoothed (about half ionized); x_ion: neutral fraction of ionized gas
  table    blackbody or grey
  tau_w    optical-depth weight (0: geometric weights); scalar: the source reading
  tuning   "" the defaults, else the autotuner's parameters for the workload
           of that name (the entries of the committed tuning cache)
"""
import functools
import math

import numpy as np
import torch

import paper_2311_01492_amd as asora

SIGMA0 = 6.3e-18
LG_LO, N_TAB, T_BB, INDEX = -20.0, 2000, 5e4, 2.8
LG_HI = {"blackbody": 4.0, "grey": math.log10(80.0)}
ALPHA_B, STEP_S = 2.59e-13, 10.0 * 3.15576e13          # case-B recombination at 1e4 K, 10 Myr
HE_EDGES, HE_LG_HI, HE_ABUNDANCE = (13.6, 24.59, 35.0, 54.42, math.inf), (2.5, 2.2, 2.3, 3.3), 0.0789

# R_whole, R_oct, max_waves, pyramid_sweep, table_place, adj_waves, adj_rate: what the
# autotuner found for 128^3 / 1000 sources / R = 30, 250^3 / 1e5 / R in [5, 50] and
# 250^3 / 1e6 / R in [5, 40]
TUNING = {"c2": (6.0, 12.0, 16, 3, 1, 16, 2), "c3": (8.0, 10.0, 12, 3, 1, 12, 2),
          "c5": (8.0, 8.0, 16, 3, 2, 16, 1)}

BASE = dict(path="forward", N=128, cell=4.3e24, n_src=1000, R_lo=30.0, R_hi=30.0, lgQ_lo=51.0, lgQ_hi=55.0,
            field="bubbles", n_bub=1000, x_ion=1e-3, table="blackbody", tau_w=0.6, scalar=False, tuning="")


def _case(name, **over):
    return dict(BASE, name=name, **over)


def listed():
    return [
        # one source in a small uniform box, with its column: the call of a script that looks at one source
        _case("column_32", path="column", N=32, n_src=1, R_lo=15.0, R_hi=15.0, lgQ_lo=54.0, lgQ_hi=54.0,
              field="uniform", n_bub=0),
        # a few small sources on an odd box through the entry point of a loop that may not allocate
        _case("static_33", path="static", N=33, n_src=5, R_lo=2.0, R_hi=12.0, n_bub=5),
        # a differentiable step of a small box, default parameters: latency and launches count
        _case("step_64", path="step", N=64, n_src=64, R_lo=20.0, R_hi=20.0, n_bub=64),
        # the rates of a thousand haloes at 30 cells on 128^3, and a differentiable step on them
        _case("forward_128", path="forward", tuning="c2"),
        _case("step_128", path="step", tuning="c2"),
        # the paper's production grid, half ionized, radii from 5 to 40: rates alone, and
        # rates with gradients where the columns do not fit in memory and are recomputed
        _case("forward_250", path="forward", N=250, cell=4.308e24, n_src=40000, R_lo=5.0, R_hi=40.0, lgQ_lo=50.0,
              lgQ_hi=54.0, field="smoothed", n_bub=0, tuning="c5"),
        _case("fwd_adj_250", path="fwd_adj", N=250, cell=4.308e24, n_src=100000, R_lo=5.0, R_hi=40.0, lgQ_lo=50.0,
              lgQ_hi=54.0, field="smoothed", n_bub=0, tuning="c5"),
        # the same grid late in reionization (almost all of it ionized), radii up to 50
        _case("fwd_adj_250_ionized", path="fwd_adj", N=250, cell=4.308e24, n_src=3000, R_lo=5.0, R_hi=50.0,
              lgQ_lo=50.0, n_bub=100000, tuning="c3"),
        # many small sources on an odd grid of highly ionized gas, default parameters
        _case("small_radii_125", path="forward", N=125, n_src=20000, R_lo=1.0, R_hi=10.0, lgQ_lo=50.0, n_bub=4000,
              x_ion=1e-5),
        # the extensions of the forward: photo-heating, and helium as a second absorber
        _case("heating_100", path="heating", N=100, n_src=500, R_lo=4.0, R_hi=28.0, n_bub=500, x_ion=1e-4),
        _case("helium_128", path="helium", N=128, n_src=300, R_lo=5.0, R_hi=20.0, n_bub=300),
        # the chemistry pass that alternates with the rates, on the production grid
        _case("chemistry_250", path="chemistry", N=250, cell=4.308e24, n_src=0, field="smoothed", n_bub=0),
    ]


# --------------------------------------------------------------------------
# Relative cost of a case: cells swept times the passes over them.
_PASSES = {"forward": 1.0, "column": 1.0, "static": 1.0, "heating": 1.5, "helium": 4.0, "fwd_adj": 4.0, "step": 3.5}


def _swept(c):
    """Sum of (4/3) pi R^3 over the sources (R uniform in [R_lo, R_hi]), at most the box each."""
    a, b = c["R_lo"], c["R_hi"]
    r3 = b ** 3 if b - a < 1e-9 else (b ** 4 - a ** 4) / (4.0 * (b - a))
    return c["n_src"] * min(4.0 / 3.0 * math.pi * r3, float(c["N"]) ** 3)


def _cost(c):
    return _PASSES.get(c["path"], 0.0) * _swept(c) + 30.0 * float(c["N"]) ** 3


def draw(rng):
    c = dict(BASE)
    log = lambda lo, hi: math.exp(rng.uniform(math.log(lo), math.log(hi)))  # noqa: E731
    c["path"] = rng.choice(["forward"] * 5 + ["fwd_adj"] * 4 + ["step"] * 3 +
                           ["column", "static", "heating", "helium", "chemistry"])
    c["N"] = min(250, int(log(16, 251)))
    if c["path"] == "static":
        c["N"] = min(64, int(log(16, 65)))
    c["cell"] = rng.choice([4.3e24, 4.308e24])
    c["R_hi"] = round(log(2.0, min(50.0, 0.6 * c["N"])), 2)
    c["R_lo"] = round(c["R_hi"] * rng.choice([1.0, 0.5, 0.1]), 2)
    c["n_src"] = 1 if c["path"] == "column" else int(log(1, 100000))
    c["lgQ_lo"] = rng.choice([50.0, 51.0])
    c["lgQ_hi"] = c["lgQ_lo"] + 4.0
    c["field"] = rng.choice(["uniform", "bubbles", "bubbles", "smoothed", "smoothed"])
    c["n_bub"] = int(log(1, 1 + c["N"] ** 3 / 160)) if c["field"] == "bubbles" else 0
    c["x_ion"] = 10.0 ** -rng.choice([3, 3, 4, 5])
    c["table"] = rng.choice(["blackbody", "blackbody", "blackbody", "grey"])
    if c["path"] in ("heating", "helium"):
        c["table"] = "blackbody"
    c["tau_w"] = rng.choice([0.6, 0.6, 0.6, 0.0])
    c["scalar"] = rng.random() < 0.2
    c["tuning"] = rng.choice(["", "", "c2", "c3", "c5"])
    if c["path"] == "chemistry":
        c["n_src"] = 0
    most = 0.6 * max(_cost(x) for x in listed())
    while c["n_src"] > 1 and _cost(c) > most:
        c["n_src"] = c["n_src"] * 2 // 3
    # kept records (about 40 bytes per swept cell at the capacity of the largest radius) stay below 20 GB
    while c["path"] == "step" and c["n_src"] > 1 and c["n_src"] * 4.2 * c["R_hi"] ** 3 * 40.0 > 2e10:
        c["n_src"] = c["n_src"] * 2 // 3
    return c


def work(case):
    n3, ns, sv = float(case["N"]) ** 3, case["n_src"], _swept(case)
    src = ns * 24.0                                     # ijk, Q, R
    path = case["path"]
    if path == "chemistry":
        return {"bytes": n3 * (4 + 4 + 8 + 8 + 8 + 8 + 4), "flops": n3 * 240.0}
    if path == "helium":
        return {"bytes": n3 * (16 + 8) + src, "flops": sv * 200.0}
    if path in ("fwd_adj", "step"):
        g = 8 if path == "fwd_adj" else 4
        return {"bytes": n3 * (8 + 4 + g + 8) + src + 8.0 * ns, "flops": sv * 210.0}
    more = {"heating": 4.0, "column": 8.0}.get(path, 0.0)
    return {"bytes": n3 * (8 + 4 + more) + src, "flops": sv * (100.0 if path == "heating" else 60.0)}


# --------------------------------------------------------------------------
# Inputs, from the seed alone.
def _device():
    return torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")


def _gaussian(N, gen, dev, sigma=None):
    """Unit-variance Gaussian field with power ~ k^-2; with sigma also a copy smoothed over sigma cells."""
    k1 = torch.fft.fftfreq(N, device=dev, dtype=torch.float64) * N
    k3 = torch.fft.rfftfreq(N, device=dev, dtype=torch.float64) * N
    k2 = k1[:, None, None] ** 2 + k1[None, :, None] ** 2 + k3[None, None, :] ** 2
    wk = torch.fft.rfftn(torch.randn((N, N, N), generator=gen, device=dev, dtype=torch.float64))
    wk = wk * torch.where(k2 > 0, k2.clamp(min=1.0) ** -0.5, torch.zeros_like(k2))
    g = torch.fft.irfftn(wk, s=(N, N, N))
    g = g / g.std()
    if sigma is None:
        return g, None
    return g, torch.fft.irfftn(wk * torch.exp(-0.5 * k2 * (2.0 * math.pi / N * sigma) ** 2), s=(N, N, N))


def _bubbles(N, centres, x_ion, gen, dev):
    """1 everywhere but in periodic balls of radius U[2, 8] around the centres."""
    x = torch.ones(N ** 3, device=dev)
    ax = torch.arange(-8, 9, device=dev)
    off = torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    d2 = (off ** 2).sum(1)
    r2 = (2.0 + 6.0 * torch.rand(centres.shape[0], generator=gen, device=dev)) ** 2
    for s in range(0, centres.shape[0], 4000):
        p = (centres[s:s + 4000, None, :].long() + off[None]) % N
        flat = (p[..., 0] * N + p[..., 1]) * N + p[..., 2]
        x[flat[d2[None].float() <= r2[s:s + 4000, None]]] = x_ion
    return x.view(N, N, N)


def _inputs(case, seed):
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 1000003 + 17)
    N, ns = case["N"], case["n_src"]
    rand = lambda n: torch.rand(n, generator=gen, device=dev, dtype=torch.float64)  # noqa: E731
    d = {}
    d["ijk"] = (rand((ns, 3)) * N).to(torch.int32).clamp(max=N - 1)
    if case["path"] == "column":
        d["ijk"][:] = N // 2
    d["Q"] = 10.0 ** (case["lgQ_lo"] + (case["lgQ_hi"] - case["lgQ_lo"]) * rand(ns))
    d["R"] = (case["R_lo"] + (case["R_hi"] - case["R_lo"]) * rand(ns)).to(torch.float32).clamp(max=case["R_hi"])
    g, gs = _gaussian(N, gen, dev, 3.0 if case["field"] == "smoothed" else None)
    if case["field"] == "uniform":
        # the seed sets the density
        d["n_H"] = torch.full((N, N, N), 1.5e-4 * math.exp(0.5 * float(g[0, 0, 0])), device=dev)
        d["x_HI"] = torch.ones((N, N, N), device=dev)
    else:
        d["n_H"] = (1.5e-4 * torch.exp(0.5 * g - 0.125)).to(torch.float32)
        if case["field"] == "smoothed":
            d["x_HI"] = torch.where(gs > gs.median(), case["x_ion"], 1.0).to(torch.float32)
        else:
            nb = case["n_bub"]
            extra = (rand((max(0, nb - ns), 3)) * N).to(torch.int32).clamp(max=N - 1)
            d["x_HI"] = _bubbles(N, torch.cat([d["ijk"][:nb], extra]), case["x_ion"], gen, dev)
    path = case["path"]
    if path == "helium":
        d["n_He"], d["x_HeI"] = HE_ABUNDANCE * d["n_H"], d["x_HI"].clone()
    if path in ("fwd_adj", "step"):
        # dL/dGamma of a loss on rates of the size these sources give a few cells away
        unit = 4.0 * math.pi * (5.0 * case["cell"]) ** 2 / (SIGMA0 * 10.0 ** (0.5 * (case["lgQ_lo"] + case["lgQ_hi"])))
        w = torch.randn((N, N, N), generator=gen, device=dev, dtype=torch.float64) * unit
        d["gbar"] = w if path == "fwd_adj" else w.to(torch.float32)
    if path == "chemistry":
        u = torch.rand((N, N, N), generator=gen, device=dev, dtype=torch.float64)
        ionized = d["x_HI"] < 0.5
        d["gamma"] = (10.0 ** torch.where(ionized, -14.0 + 2.5 * u, -18.0 + 3.0 * u)).to(torch.float32)
        d["y0"] = torch.where(ionized, 10.0 ** (-4.0 + 2.0 * u), 1.0 - 0.05 * u)
    return d


# --------------------------------------------------------------------------
# What the program holds, and one pass.
@functools.lru_cache(maxsize=None)
def _host_table(kind):
    if kind == "grey":
        return asora.table_grey(N_TAB, LG_LO, LG_HI["grey"])
    if kind == "heat":
        return asora.table_blackbody_heat(T_BB, INDEX, N_TAB, LG_LO, LG_HI["blackbody"])
    if kind.startswith("band"):
        b = int(kind[4:])
        return asora.table_blackbody_band(HE_EDGES[b], HE_EDGES[b + 1], T_BB, INDEX, N_TAB, LG_LO, HE_LG_HI[b])
    return asora.table_blackbody(T_BB, INDEX, N_TAB, LG_LO, LG_HI["blackbody"])


def _he_sections():
    sH = [SIGMA0 * (e / 13.6) ** -2.8 for e in HE_EDGES[:-1]]
    r = [e / 24.59 for e in HE_EDGES[:-1]]
    return sH, [7.42e-18 * (1.66 * x ** -2.05 - 0.66 * x ** -3.05) if x >= 1.0 else 0.0 for x in r]


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case, path=case["path"], R_max=float(case["R_hi"]))
    N, path = case["N"], case["path"]
    P, dP = _host_table(case["table"])
    ctx = asora.Asora(N, case["cell"], P, dP, lg_lo=LG_LO, lg_hi=LG_HI[case["table"]],
                      tau_w=case["tau_w"] if case["tau_w"] > 0 else math.inf, halfpath_scalar=case["scalar"])
    if case["tuning"]:
        ctx.set_tuning(*TUNING[case["tuning"]])
    s["ctx"] = ctx
    dev = s["n_H"].device
    grid = lambda dt: torch.empty((N, N, N), dtype=dt, device=dev)  # noqa: E731
    if path in ("forward", "static", "heating", "helium", "fwd_adj"):
        s["out"] = grid(torch.float32)
    if path == "heating":
        ctx.set_heating_table(*_host_table("heat"))
        s["out2"] = grid(torch.float32)
    if path == "helium":
        sH, sHe = _he_sections()
        ctx.set_helium([_host_table("band%d" % b) + (LG_LO, HE_LG_HI[b], sH[b], sHe[b]) for b in range(4)])
        s["out2"] = grid(torch.float32)
    if path == "fwd_adj":
        s["grads"] = (grid(torch.float32), grid(torch.float32),
                      torch.empty(case["n_src"], dtype=torch.float64, device=dev))
    if path == "step":
        for k in ("n_H", "x_HI", "Q"):
            s[k].requires_grad_(True)
    if path == "chemistry":
        # the pass before this one: the same gas in a rate that was 10 % lower
        s["prev"] = ctx.chemistry(0.9 * s["gamma"], s["n_H"], s["y0"], STEP_S, ALPHA_B)[0]
    return s


def run(s):
    ctx, path = s["ctx"], s["path"]
    if path == "chemistry":
        y_avg, y_end, y32, changed = ctx.chemistry(s["gamma"], s["n_H"], s["y0"], STEP_S, ALPHA_B,
                                                   xHI_avg_prev=s["prev"])
        return {"y_avg": y_avg, "y_end": y_end, "y32": y32, "changed": changed}
    src = (s["ijk"], s["Q"], s["R"])
    if path == "column":
        gamma, cd = ctx.raytrace(s["n_H"], s["x_HI"], *src, R_max=s["R_max"], coldens=True)
        return {"gamma": gamma, "column": cd}
    if path == "static":
        return {"gamma": ctx.raytrace_static(s["n_H"], s["x_HI"], *src, R_max=s["R_max"], out=s["out"])}
    if path == "heating":
        gamma, heat = ctx.raytrace_heating(s["n_H"], s["x_HI"], *src, R_max=s["R_max"], out=s["out"],
                                           heating_out=s["out2"])
        return {"gamma": gamma, "heating": heat}
    if path == "helium":
        gH, gHe = ctx.raytrace_helium(s["n_H"], s["x_HI"], s["n_He"], s["x_HeI"], *src, R_max=s["R_max"],
                                      out=(s["out"], s["out2"]))
        return {"gamma": gH, "gamma_he": gHe}
    if path == "step":
        for k in ("n_H", "x_HI", "Q"):
            s[k].grad = None
        gamma = asora.raytrace(ctx, s["n_H"], s["x_HI"], *src, R_max=s["R_max"])
        gamma.backward(s["gbar"])
        return {"gamma": gamma.detach(), "dn": s["n_H"].grad, "dx": s["x_HI"].grad, "dq": s["Q"].grad}
    gamma = ctx.raytrace(s["n_H"], s["x_HI"], *src, R_max=s["R_max"], out=s["out"])
    if path == "forward":
        return {"gamma": gamma}
    dn, dx, dq = ctx.backward(s["n_H"], s["x_HI"], *src, s["gbar"], R_max=s["R_max"], out=s["grads"])
    return {"gamma": gamma, "dn": dn, "dx": dx, "dq": dq}


# --------------------------------------------------------------------------
# The same outputs in float64 torch, straight from the formulas: shells of
# equal largest offset m, every shell's entry columns interpolated from the
# four cells of shell m - 1 next to it, all sources of a batch at once.
@functools.lru_cache(maxsize=None)
def _table64(kind):
    """(lg_lo, lg_hi, ln P, d ln P / d ln tau, P_0, P'_0) by quadrature in ln x."""
    band = int(kind[4:]) if kind.startswith("band") else -1
    lg_hi = HE_LG_HI[band] if band >= 0 else LG_HI["grey" if kind == "grey" else "blackbody"]
    tau = 10.0 ** np.linspace(LG_LO, lg_hi, N_TAB)
    if kind == "grey":
        P, dP = np.exp(-tau), -np.exp(-tau)
    else:
        kT = 8.617333262e-5 * T_BB
        x0 = 13.6 / kT
        nodes, weights = np.polynomial.legendre.leggauss(24)

        def rule(a, b, panels=160):
            e = np.linspace(math.log(a), math.log(b), panels + 1)
            h = 0.5 * np.diff(e)[:, None]
            x = np.exp(0.5 * (e[1:] + e[:-1])[:, None] + h * nodes[None, :])
            return x.reshape(-1), (h * weights[None, :] * x).reshape(-1)

        photons = lambda x: x * x * np.exp(-x) / -np.expm1(-x)  # noqa: E731
        x, w = rule(x0, 800.0)
        norm = float(np.sum(w * photons(x)))
        xa, xb = (x0, 800.0) if band < 0 else (HE_EDGES[band] / kT, min(HE_EDGES[band + 1] / kT, 800.0))
        x, w = rule(xa, xb)
        w = w * photons(x) * ((x - x0) * kT if kind == "heat" else 1.0) / norm
        shape = (x / xa) ** -INDEX
        P, dP = np.empty(N_TAB), np.empty(N_TAB)
        for t in range(N_TAB):
            e = w * np.exp(-tau[t] * shape)
            P[t], dP[t] = e.sum(), -(e * shape).sum()
    return LG_LO, lg_hi, np.log(P), tau * dP / P, float(P[0]), float(dP[0])


class _Table:
    def __init__(self, kind, dev):
        lo, hi, y, m, self.P0, self.dP0 = _table64(kind)
        self.x_lo, self.n = lo * math.log(10.0), N_TAB
        self.h = (hi - lo) * math.log(10.0) / (N_TAB - 1)
        self.y, self.m = torch.as_tensor(y, device=dev), torch.as_tensor(m, device=dev)
        self.tau_lo, self.tau_hi = math.exp(self.x_lo), math.exp(self.x_lo + self.h * (N_TAB - 1))
        self.P_hi = math.exp(float(y[-1]))

    def P(self, tau):
        inside = tau.clamp(self.tau_lo, self.tau_hi)
        t = (torch.log(inside) - self.x_lo) / self.h
        j = t.detach().floor().long().clamp(0, self.n - 2)
        f = t - j
        y0, y1, a, b = self.y[j], self.y[j + 1], self.h * self.m[j], self.h * self.m[j + 1]
        d = y1 - y0
        p = torch.exp(y0 + f * (a + f * (3 * d - 2 * a - b + f * (a + b - 2 * d))))
        p = torch.where(tau < self.tau_lo, self.P0 + self.dP0 * (tau - self.tau_lo), p)
        return torch.where(tau >= self.tau_hi, torch.full_like(p, self.P_hi), p)

    def absorbed(self, tau, dtau):
        """-[P(tau + dtau) - P(tau)] / dtau."""
        return (self.P(tau) - self.P(tau + dtau)) / dtau


def _shells(N, Rsq, dev):
    """Per shell m: offsets [n, 3], r^2 [n] (ascending), indices [4, n] into shell m - 1 and geometric weights."""
    neg = N // 2 if N % 2 == 0 else (N - 1) // 2
    pos = N // 2 - 1 if N % 2 == 0 else (N - 1) // 2
    M = min(math.isqrt(Rsq), neg)
    ax = torch.arange(-M, M + 1, device=dev)
    off = torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    r2 = (off ** 2).sum(1)
    off = off[(r2 <= Rsq) & (off <= pos).all(1) & (off >= -neg).all(1)]
    r2 = (off ** 2).sum(1)
    order = torch.argsort(r2, stable=True)
    off, r2 = off[order], r2[order]
    mm = off.abs().max(1).values
    side = 2 * M + 1
    where = torch.zeros(side ** 3, dtype=torch.long, device=dev)
    flat = lambda o: ((o[..., 0] + M) * side + o[..., 1] + M) * side + o[..., 2] + M  # noqa: E731
    shells = []
    for m in range(1, M + 1):
        o = off[mm == m]
        a = o.abs()
        d = a.argmax(1)
        i = torch.arange(o.shape[0], device=dev)
        u, v = torch.where(d == 0, 1, 0), torch.where(d == 2, 1, 2)
        sg = torch.sign(o)
        idx, wt = [], []
        for su, sv in ((0, 0), (1, 0), (0, 1), (1, 1)):
            e = o.clone()
            e[i, d] -= sg[i, d]
            if su:
                e[i, u] -= sg[i, u]
            if sv:
                e[i, v] -= sg[i, v]
            fu, fv = a[i, u].double() / m, a[i, v].double() / m
            w = (fu if su else 1 - fu) * (fv if sv else 1 - fv)
            idx.append(torch.where(w > 0, where[flat(e)], torch.zeros_like(i)))
            wt.append(w)
        shells.append((o, r2[mm == m], torch.stack(idx), torch.stack(wt)))
        where[flat(o)] = i
    return shells


def _trace64(case, d, species, tables, rate, grads=None):
    """Adds every source's rate to grids: `species` the densities whose columns are carried (the first sets the
    weights), rate(columns, in-cell columns) the rates per (Q / 4 pi alpha^2 r^2), one output grid per value."""
    N, alpha, dev = case["N"], case["cell"], d["n_H"].device
    tw, reading = case["tau_w"], 1 if case["scalar"] else 0
    Rsq = torch.floor(d["R"].double() ** 2).long()
    order = torch.argsort(Rsq)
    shells = _shells(N, int(Rsq.max()) if Rsq.numel() else 0, dev)
    n_out = len(rate([torch.zeros(1, dtype=torch.float64, device=dev) + 1e10] * len(species),
                     [torch.zeros(1, dtype=torch.float64, device=dev) + 1e10] * len(species)))
    out = [torch.zeros(N ** 3, dtype=torch.float64, device=dev) for _ in range(n_out)]
    column = torch.zeros(N ** 3, dtype=torch.float64, device=dev)
    room = 3e7 if grads is None else 1e7   # cells in flight
    lo = 0
    while lo < order.numel():
        # a batch of sources of like radii
        hi = lo
        while hi < order.numel():
            step = max(1, min(4096, order.numel() - hi))
            top = float(Rsq[order[min(order.numel(), hi + step) - 1]])
            while step > 1 and (hi + step - lo) * 4.2 * top ** 1.5 > room:
                step //= 2
                top = float(Rsq[order[hi + step - 1]])
            if hi > lo and (hi + step - lo) * 4.2 * top ** 1.5 > room:
                break
            hi += step
        k = order[lo:hi]
        lo = hi
        src, Q, rs = d["ijk"][k].long(), d["Q"][k].double(), Rsq[k]
        if grads is not None:
            Q = Q.requires_grad_(True)
        top = int(rs.max())
        cs = (src[:, 0] * N + src[:, 1]) * N + src[:, 2]
        half = [s.index_select(0, cs) * alpha * 0.5 for s in species]
        zero = [torch.zeros_like(h) for h in half]
        parts = [(cs, [g * Q / (2 * alpha ** 2) for g in rate(zero, half)])]
        prev = None
        for m, (o, r2, idx, wt) in enumerate(shells, 1):
            n = int(torch.searchsorted(r2, top, right=True))
            if n == 0:
                break
            o, r2, idx, wt = o[:n], r2[:n], idx[:, :n], wt[:, :n]
            ds = torch.sqrt(r2.double()) / m
            w3 = [(src[:, ax, None] + o[None, :, ax]) % N for ax in range(3)]
            cp = ((w3[0] * N + w3[1]) * N + w3[2]).reshape(-1)
            dN = [s.index_select(0, cp).reshape(len(k), n) * (alpha * ds)[None] for s in species]
            if m == 1:
                Nin = [h[:, None] * (ds[None] if reading == 0 else torch.ones_like(ds)[None]) for h in half]
            else:
                W, num = 0.0, [0.0] * len(species)
                for q in range(4):
                    M = [p.index_select(1, idx[q]) for p in prev]
                    w = wt[q][None] / (SIGMA0 * M[0]).clamp(min=tw) if tw > 0 else wt[q][None]
                    W = W + w
                    num = [a + w * b for a, b in zip(num, M)]
                Nin = [a / W for a in num]
            prev = [a + b for a, b in zip(Nin, dN)]
            mask = (r2[None] <= rs[:, None]).double()
            scale = Q[:, None] / (4 * math.pi * alpha ** 2 * r2.double())[None] * mask
            parts.append((cp, [(g * scale).reshape(-1) for g in rate(Nin, dN)]))
            if case["path"] == "column":
                column.index_add_(0, cp, (Nin[0] * mask).reshape(-1).detach())
        for cp, gs in parts:
            for g, acc in zip(gs, out):
                acc.index_add_(0, cp, g.detach())
        if grads is not None:
            loss = sum((gs[0] * grads["gbar"].index_select(0, cp)).sum() for cp, gs in parts)
            gn, gq = torch.autograd.grad(loss, [species[0], Q])
            grads["nbar"] += gn
            grads["dq"][k] = gq
    return out, column


def exact(case, seed):
    grad = case["path"] in ("fwd_adj", "step")
    if _swept(case) * (8.0 if grad else 3.0 if case["path"] == "helium" else 1.0) > 4e9:
        return None   # tens of seconds
    d = _inputs(case, seed)
    dev, N, path = d["n_H"].device, case["N"], case["path"]
    shape = (N, N, N)
    if path == "chemistry":
        g, nH, y0 = d["gamma"].double(), d["n_H"].double(), d["y0"]
        y = y0.clone()
        for _ in range(100):
            rate = g + nH * (1.0 - y) * ALPHA_B
            u, eq = rate * STEP_S, torch.where(rate > 0, nH * (1.0 - y) * ALPHA_B / rate, torch.ones_like(rate))
            new = eq + (y0 - eq) * torch.where(u > 0, -torch.expm1(-u) / u, torch.ones_like(u))
            end = eq + (y0 - eq) * torch.exp(-u)
            moved = bool(((new - y).abs() > 1e-13 * new).any())
            y = new
            if not moved:
                break
        return {"y_avg": y, "y_end": end, "y32": y, "changed": None}
    n_H, x_HI = d["n_H"].double().reshape(-1), d["x_HI"].double().reshape(-1)
    species, tables = [n_H * x_HI], [_Table(case["table"], dev)]
    rate = lambda N_, dN: [SIGMA0 * tables[0].absorbed(SIGMA0 * N_[0], SIGMA0 * dN[0])]  # noqa: E731
    if path == "heating":
        tables.append(_Table("heat", dev))
        rate = lambda N_, dN: [SIGMA0 * t.absorbed(SIGMA0 * N_[0], SIGMA0 * dN[0]) for t in tables]  # noqa: E731
    if path == "helium":
        species.append(d["n_He"].double().reshape(-1) * d["x_HeI"].double().reshape(-1))
        tables = [_Table("band%d" % b, dev) for b in range(4)]
        sH, sHe = _he_sections()

        def rate(N_, dN):
            D = [t.absorbed(a * N_[0] + b * N_[1], a * dN[0] + b * dN[1]) for t, a, b in zip(tables, sH, sHe)]
            return [sum(a * x for a, x in zip(sH, D)), sum(b * x for b, x in zip(sHe, D))]

    if not grad:
        with torch.no_grad():
            out, column = _trace64(case, d, species, tables, rate)
        out = [o.view(shape) for o in out]
        if path == "column":
            return {"gamma": out[0], "column": column.view(shape)}
        if path == "heating":
            return {"gamma": out[0], "heating": out[1]}
        if path == "helium":
            return {"gamma": out[0], "gamma_he": out[1]}
        return {"gamma": out[0]}
    species = [species[0].requires_grad_(True)]
    gr = {"gbar": d["gbar"].double().reshape(-1), "nbar": torch.zeros_like(n_H),
          "dq": torch.zeros(case["n_src"], dtype=torch.float64, device=dev)}
    out, _ = _trace64(case, d, species, tables, rate, gr)
    return {"gamma": out[0].view(shape), "dn": (x_HI * gr["nbar"]).view(shape), "dx": (n_H * gr["nbar"]).view(shape),
            "dq": gr["dq"]}
