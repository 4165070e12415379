"""The work that a user of this library has it do, as a list of cases to time.

listed()   the cases;
draw(rng)  one more case of the same ranges;
prepare()  what a program holds before the call: the loaded model, the call's
           parameters and, where it keeps them, its output buffers;
run()      one pass through the public entry points;
work()     the bytes and operations that the pass cannot do without;
exact()    the same outputs from torch in 64 bits, without the library.

The models are the seeded ones of synth/ (no first-principles data is
available); Fermi level, temperatures, the k points of a subset and, for the
small models, the vertex g follow the seed.  A program loads a model once and
makes many calls with it, so a loaded model is kept for later calls.

Rates of the reduced-precision forms are returned in 32 bits, which is what
those forms compute in; energies and velocities are FP64 in every form.
"""
from __future__ import annotations

import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2306_16493_amd import Context
from paper_2306_16493_amd.eph import Mlp
from synth import WORKLOADS, make_system

_WORKLOAD = {"toy_sc": "toy_sc_8", "al_fcc": "al_fcc_100", "si_fcc": "si_fcc_150"}
_SHAPE = {  # orbitals, modes, electron and phonon lattice vectors of g
    "toy_sc": (4, 3, 64, 64), "al_fcc": (4, 3, 216, 216), "si_fcc": (8, 6, 512, 216)}
# share of the N^3 N_w (k, band) states inside the window, and vertices per
# (state, q) pair, of the models (from the library's own counts)
_DENSITY = {"toy_sc": (1.0, 1.0), "al_fcc": (0.109, 0.22), "si_fcc": (0.037, 0.16)}
_WIDTH = 128  # hidden units of the surrogate network (three layers), 10 inputs


def listed():
    rates = dict(kind="rates", subset=1.0, n_temps=1, keep=False)
    return [
        # the smallest run: every state of the toy model on 8^3 grids; latency and launches
        dict(rates, name="toy 8 fp64", system="toy_sc", grid=8, precision="fp64"),
        # a convergence-study point of a metal: coarse grid, three temperatures, FP64
        dict(rates, name="al 24 fp64", system="al_fcc", grid=24, precision="fp64", n_temps=3),
        # the same on a finer grid in the split-bf16 form
        dict(rates, name="al 36 bf16x3", system="al_fcc", grid=36, precision="bf16x3", n_temps=3),
        # a share of the production grid in FP64, as one worker of many has it;
        # sized once, buffers kept
        dict(rates, name="al 100 fp64 part", system="al_fcc", grid=100, precision="fp64", n_temps=3, subset=0.04,
             keep=True),
        # a whole production run of the metal, the headline form, on an odd-sized grid
        dict(rates, name="al 71 bf16x3", system="al_fcc", grid=71, precision="bf16x3", n_temps=3, keep=True),
        # scattered training k points of the surrogate on a large grid
        dict(rates, name="al 160 fp32 part", system="al_fcc", grid=160, precision="fp32", subset=0.0025),
        # the semiconductor (8 orbitals, 6 modes), FP64
        dict(rates, name="si 48 fp64 part", system="si_fcc", grid=48, precision="fp64", subset=0.08),
        # the semiconductor on a production grid: large tables, long lines, few states
        dict(rates, name="si 130 fp32 part", system="si_fcc", grid=130, precision="fp32", subset=0.0015),
        # transition rates and ten iterations of the Boltzmann equation
        dict(kind="bte", name="al 18 iterative", system="al_fcc", grid=18, n_temps=2, iterations=10),
        # the surrogate's fit (a stretch of its 30000 steps) and its inference for every state
        dict(kind="train", name="surrogate fit", samples=70000, members=5, n_out=1, batch=512, steps=60),
        dict(kind="predict", name="surrogate predict", samples=437296, members=5, n_out=1),
        # conductivity, Seebeck and electronic thermal conductivity of a finished run
        dict(kind="transport", name="transport", samples=437296, n_temps=3),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


# pass cost of a rates call in (state, q) pairs of the Al-like model in FP32:
# FP64 costs about twice, a Si-like pair about five times as much
_COST = {"toy_sc": 3.0, "al_fcc": 1.0, "si_fcc": 5.0}
_MOST = 4.5e10


def draw(rng):
    kind = rng.choice(["rates"] * 8 + ["bte", "train", "predict", "transport"])
    if kind == "train":
        return dict(kind=kind, samples=int(_log(rng, 2000, 200000)), members=rng.randint(1, 8), n_out=rng.randint(1, 4),
                    batch=32 * int(_log(rng, 1, 33)), steps=rng.randint(20, 100))
    if kind == "predict":
        return dict(kind=kind, samples=int(_log(rng, 500, 1500000)), members=rng.randint(1, 8), n_out=rng.randint(1, 4))
    if kind == "transport":
        return dict(kind=kind, samples=int(_log(rng, 500, 4000000)), n_temps=rng.randint(1, 4))
    if kind == "bte":
        system = rng.choice(["toy_sc", "al_fcc"])
        grid = rng.randint(4, 11) if system == "toy_sc" else rng.randint(8, 26)
        return dict(kind=kind, system=system, grid=grid, n_temps=rng.randint(1, 4), iterations=rng.randint(3, 20))
    system = rng.choice(["toy_sc", "al_fcc", "al_fcc", "al_fcc", "si_fcc", "si_fcc"])
    lo, hi = {"toy_sc": (4, 16), "al_fcc": (12, 160), "si_fcc": (10, 130)}[system]
    grid = int(round(_log(rng, lo, hi)))
    precision = rng.choice(["fp64", "fp32", "bf16x3"])
    most = _MOST / _COST[system] / (2.0 if precision == "fp64" else 1.0) / grid ** 3  # states
    states = _DENSITY[system][0] * _SHAPE[system][0] * grid ** 3
    subset = 1.0 if rng.random() < 0.4 else _log(rng, 0.002, 0.5)
    subset = max(min(subset, 0.8 * most / states), min(1.0, 100.0 / states))
    return dict(kind="rates", system=system, grid=grid, precision=precision, n_temps=rng.randint(1, 4),
                subset=float("%.3g" % subset) if subset < 1.0 else 1.0, keep=rng.random() < 0.5)


# ---------------------------------------------------------------- inputs

@functools.lru_cache(maxsize=None)
def _system(name, variant):
    s = make_system(name)
    return dataclasses.replace(s, gw=make_system(name, seed=7000 + variant).gw) if variant else s


@functools.lru_cache(maxsize=None)
def _context(name, variant):
    return Context(_system(name, variant), device=0)


def _variant(name, seed):
    return 0 if name == "si_fcc" else seed % 3  # the Si-like g is 680 MB: one of it


@functools.lru_cache(maxsize=None)
def _band_edge(name, variant, grid):
    """Lowest energy of the first conduction band on the grid."""
    w = WORKLOADS[_WORKLOAD[name]]
    ctx = _context(name, variant)
    p = ctx.params(grid, 0.0, [300.0], w.eta, -1e6, 1e6, band_lo=w.band_lo, band_hi=w.band_lo)
    return float(ctx.select_states(p)[2].min().item())


def _window(name, grid):
    """Reference level (band centroid, or lowest conduction energy on the grid) and state window."""
    w = WORKLOADS[_WORKLOAD[name]]
    if w.window_relative_to == "mu":
        level = _system(name, 0).mu_centroid
        return w, level, level + w.window[0], level + w.window[1]
    level = _band_edge(name, 0, grid)
    return w, level, level + w.window[0] - 1e-7, level + w.window[1]


def _conditions(case, seed):
    """Model, Fermi level, window and temperatures of a call."""
    w, level, lo, hi = _window(case["system"], case["grid"])
    rng = np.random.default_rng([seed, 11])
    base = {1: [300.0], 2: [200.0, 300.0], 3: [100.0, 300.0, 500.0], 4: [100.0, 200.0, 300.0, 500.0]}[case["n_temps"]]
    temps = [t * float(rng.uniform(0.95, 1.05)) for t in base]
    mu = level + (0.0 if w.window_relative_to == "mu" else -0.25) + float(rng.uniform(-0.02, 0.02))
    return w, _variant(case["system"], seed), mu, lo, hi, temps


@functools.lru_cache(maxsize=None)
def _states_per_k(name, grid):
    """(k points with states in the window, states of each)."""
    w, level, lo, hi = _window(name, grid)
    ctx = _context(name, 0)
    p = ctx.params(grid, level, [300.0], w.eta, lo, hi, w.band_lo, w.band_hi)
    return np.unique(ctx.select_states(p)[0].cpu().numpy().astype(np.int64), return_counts=True)


def _subset(case, seed):
    """A random choice of k points that carry a given share of the window's states; None for all."""
    if case.get("subset", 1.0) >= 1.0:
        return None
    k, count = _states_per_k(case["system"], case["grid"])
    want = max(1, int(round(case["subset"] * int(count.sum()))))
    at = np.random.default_rng([seed, 12]).permutation(k.size)
    n = int(np.searchsorted(np.cumsum(count[at]), want, side="right"))
    short = want - int(count[at[:n]].sum())
    rest = at[n:]
    return np.sort(np.concatenate([k[at[:n]], k[rest[count[rest] == 1][:short]]]))


def _samples(case, seed):
    """Features-like inputs and log-rate-like targets of the surrogate, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, nout = case["samples"], case["n_out"]
    r = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float64)
    ang = 2.0 * math.pi * r(n, 3)
    x = torch.empty(n, 10, dtype=torch.float64, device="cuda")
    x[:, 0:6:2], x[:, 1:6:2] = torch.sin(ang), torch.cos(ang)
    x[:, 6] = 0.6 * r(n) - 0.3
    x[:, 7:] = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64) * 0.4
    y = torch.empty(n, nout, dtype=torch.float64, device="cuda")
    for t in range(nout):
        y[:, t] = 30.0 + 0.3 * t + 0.5 * torch.sin(ang[:, 0]) * torch.cos(ang[:, 1]) + x[:, 6] + 0.1 * x[:, 7:].sum(1)
    return x.float().contiguous(), y.float().contiguous()


def _weights(case, seed):
    """Parameters W1 b1 W2 b2 W3 b3 W4 b4 of every member, FP32."""
    rng = np.random.default_rng([seed, 13])
    out = []
    for _ in range(case["members"]):
        for fan_in, fan_out in ((10, _WIDTH), (_WIDTH, _WIDTH), (_WIDTH, _WIDTH), (_WIDTH, case["n_out"])):
            out.append(rng.uniform(-1.0, 1.0, fan_out * fan_in) * math.sqrt(3.0 / fan_in))
            out.append(rng.uniform(-0.1, 0.1, fan_out))
    return np.concatenate(out).astype(np.float32).reshape(case["members"], -1)


def _state_arrays(case, seed):
    """Energies, velocities and rates of a finished run, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, nt = case["samples"], case["n_temps"]
    r = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float64)
    e = 0.6 * r(n) - 0.3 + 1.25
    v = 4e5 * torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    it = torch.exp(30.0 + torch.randn(nt, n, generator=g, device="cuda", dtype=torch.float64))
    return e, v, it, 1.25 + 0.01 * (seed % 5), [150.0 + 90.0 * t for t in range(nt)]


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind in ("rates", "bte"):
        w, variant, mu, lo, hi, temps = _conditions(case, seed)
        ctx = _context(case["system"], variant)
        st.update(ctx=ctx, mu=mu, temps=temps, cells=case["grid"] ** 3, buffers=None, capacity=None)
        st["params"] = ctx.params(case["grid"], mu, temps, w.eta, lo, hi, w.band_lo, w.band_hi,
                                  precision=case.get("precision", "fp64"), k_subset=_subset(case, seed))
        if case.get("keep"):
            n = ctx.count_states(st["params"])
            cap = max(n, 1)
            st["capacity"] = n
            st["buffers"] = dict(k=torch.empty(cap, dtype=torch.int32, device="cuda"),
                                 n=torch.empty(cap, dtype=torch.int32, device="cuda"),
                                 e=torch.empty(cap, dtype=torch.float64, device="cuda"),
                                 v=torch.empty(cap, 3, dtype=torch.float64, device="cuda"),
                                 it=torch.empty(len(temps) * cap, dtype=torch.float64, device="cuda"))
    elif kind == "train":
        st["x"], st["y"] = _samples(case, seed)
        st["mlp"] = Mlp(_context("toy_sc", 0), members=case["members"], n_out=case["n_out"], seed=seed)
    elif kind == "predict":
        st["x"], y = _samples(case, seed)
        st["mlp"] = Mlp(_context("toy_sc", 0), members=case["members"], n_out=case["n_out"], seed=seed)
        st["mlp"].train(st["x"], y, steps=1, batch=32)  # fixes the normalisation
        st["mlp"].set_params(_weights(case, seed))
    else:
        st["ctx"] = _context("toy_sc", 0)
        st["arrays"] = _state_arrays(case, seed)
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "rates":
        ctx = st["ctx"]
        res, _ = ctx.scattering_rates(st["params"], capacity=st["capacity"], buffers=st["buffers"])
        sig = ctx.conductivity(res.energy, res.vel, res.inv_tau.reshape(-1), st["mu"], st["temps"], st["cells"])
        it = res.inv_tau
        if case["precision"] != "fp64":
            it, sig = it.float(), sig.astype(np.float32)
        return dict(k=res.state_k, n=res.state_n, energy=res.energy, vel=res.vel, inv_tau=it, sigma=sig,
                    counts=res.counts)
    if kind == "bte":
        ctx = st["ctx"]
        res, gamma = ctx.rates_gamma(st["params"])
        sig, done, F = ctx.bte_iterate(gamma, res, st["cells"], max_iter=case["iterations"], tol=0.0, want_f=True)
        info = gamma.info()
        gamma.close()
        return dict(k=res.state_k, n=res.state_n, inv_tau=res.inv_tau, sigma=sig, F=F, iterations=done,
                    entries=info["nnz"], bytes=info["bytes"])
    if kind == "train":
        loss = st["mlp"].train(st["x"], st["y"], steps=case["steps"], batch=case["batch"], lr=2e-3)
        return dict(loss=loss, params=st["mlp"].get_params())
    if kind == "predict":
        return dict(y=st["mlp"].predict(st["x"]))
    e, v, it, mu, temps = st["arrays"]
    sig, see, kap = st["ctx"].transport(e, v, it, mu, temps, 10 ** 6)
    return dict(sigma=sig, seebeck=see, kappa=kap)


# ---------------------------------------------------------------- work

def work(case):
    kind = case["kind"]
    P = 10 * _WIDTH + _WIDTH + 2 * (_WIDTH * _WIDTH + _WIDTH) + case.get("n_out", 1) * (_WIDTH + 1)
    if kind == "train":  # three products (forward, input and weight gradient) per weight and sample
        it = case["members"] * case["steps"]
        return dict(flops=6.0 * P * it * case["batch"],
                    bytes=4.0 * case["samples"] * (10 + case["n_out"]) + 2 * 12.0 * case["members"] * P)
    if kind == "predict":
        return dict(flops=2.0 * P * case["members"] * case["samples"],
                    bytes=4.0 * case["samples"] * (10 + case["members"] * case["n_out"]))
    if kind == "transport":  # three moments of nine elements per state and temperature
        return dict(flops=case["samples"] * case["n_temps"] * 60.0,
                    bytes=8.0 * case["samples"] * (4 + case["n_temps"]))
    nw, nm, nre, nrp = _SHAPE[case["system"]]
    share, hits = _DENSITY[case["system"]]
    edge = round(nrp ** (1 / 3))
    N = case["grid"]
    states = max(1.0, share * nw * N ** 3 * case.get("subset", 1.0))
    C = nw * nm
    flops = 8.0 * states * (nre * nw * nrp * C                 # Re transform
                            + N * nrp * C + N * N * edge ** 2 * C  # separable Rp sum
                            + hits * N ** 3 * (edge * C + edge * nm + nm * nm))
    eig = 8.0 * N ** 3 * (12 * nw ** 3 + 12 * nm ** 3)  # band and mode tables
    # model read once; band energies, velocities and eigenvectors, mode
    # energies and matrices written and read once; outputs written once
    nbytes = 16.0 * nre * nrp * C * nw + 2 * N ** 3 * (nw * (8 + 24 + 16 * nw) + nm * (8 + 16 * nm))
    nbytes += states * (4 + 4 + 8 + 24 + 8 * case["n_temps"])
    if kind == "bte":  # transition rates written once and read in every iteration
        entries = states * states * hits * 0.5
        nbytes += entries * (4 + 8 * case["n_temps"]) * (1 + case["iterations"])
        flops += 6.0 * entries * case["n_temps"] * case["iterations"]
    return dict(flops=flops + eig, bytes=nbytes)


# ---------------------------------------------------------------- 64-bit values

_H, _E, _KB, _AMU = 6.62607015e-34, 1.602176634e-19, 1.380649e-23, 1.66053906892e-27
_HBAR = _H / (2.0 * math.pi)


def _to_grid(vecs, vals, N):
    """sum_R e^{i k.R} vals[R] on the N^3 grid: [N^3, ...], index i1 + N (i2 + N i3)."""
    r = torch.as_tensor(np.mod(np.asarray(vecs, np.int64), N), device="cuda")
    idx = r[:, 0] + N * (r[:, 1] + N * r[:, 2])
    flat = vals.reshape(vals.shape[0], -1)
    box = torch.zeros(N ** 3, flat.shape[1], dtype=torch.complex128, device="cuda")
    box.index_add_(0, idx, flat)
    out = torch.fft.ifftn(box.view(N, N, N, -1), dim=(0, 1, 2), norm="forward")
    return out.reshape((N ** 3,) + tuple(vals.shape[1:]))


def _eigh(m):
    w, v = torch.linalg.eigh(m.cpu())
    return w.cuda(), v.cuda()


def _exact_tables(s, N, omega_cut=1e-4):
    c = lambda a: torch.as_tensor(np.asarray(a), device="cuda").to(torch.complex128)
    wh = c(s.rh_w)[:, None, None] * c(s.ham)
    eps, V = _eigh(_to_grid(s.rh, wh, N))                 # V[k][i][n]
    cart = s.rh @ s.lattice
    vel = torch.empty(N ** 3, s.nw, 3, dtype=torch.float64, device="cuda")
    for a in range(3):
        d = _to_grid(s.rh, 1j * c(cart[:, a])[:, None, None] * wh, N)
        vel[:, :, a] = (V.conj() * _small(d, V)).sum(1).real * (_E * 1e-10 / _HBAR)
    mass = np.repeat(np.asarray(s.mass), 3)
    dyn = c(s.rd_w)[:, None, None] * c(s.ifc / np.sqrt(mass[:, None] * mass[None, :]))
    lam, e = _eigh(_to_grid(s.rd, dyn, N))
    cph = _HBAR * _HBAR / (_AMU * 1e-20) / _E
    om = torch.sqrt(cph * torch.clamp(lam, min=0.0))
    live = om >= omega_cut
    amp = torch.sqrt(cph / (2.0 * torch.as_tensor(mass, device="cuda")[None, :, None] * om.clamp(min=1e-30)[:, None, :]))
    u = torch.where(live[:, None, :], e * amp, torch.zeros((), dtype=torch.complex128, device="cuda"))  # u[q][mu][nu]
    return eps, V, vel, om, u, live


def _small(a, b):
    """Batched product of small matrices by elementwise sums."""
    out = torch.zeros(a.shape[:-1] + b.shape[-1:], dtype=a.dtype, device=a.device)
    for i in range(a.shape[-1]):
        out += a[..., :, i, None] * b[..., i, None, :]
    return out


def _exact_states(case, seed, s, tables, w, lo, hi):
    eps = tables[0]
    nb = s.nw - 1 if w.band_hi < 0 else w.band_hi
    ok = (eps >= lo) & (eps <= hi)
    band = torch.arange(s.nw, device="cuda")
    ok &= ((band >= w.band_lo) & (band <= nb))[None, :]
    ks = _subset(case, seed)
    if ks is not None:
        m = torch.zeros(case["grid"] ** 3, dtype=torch.bool, device="cuda")
        m[torch.as_tensor(ks, device="cuda")] = True
        ok &= m[:, None]
    k, n = ok.nonzero(as_tuple=True)
    return k, n


def _exact_rates(s, N, w, tables, k, n, mu, temps, gamma_rows=None):
    """1/tau [nt][ns]; gamma_rows(s0, rows [b][m][N^3 final k][nt]) receives the
    transition rates of each batch of states."""
    eps, V, vel, om, u, live = tables
    nw, nm, ns, nt = s.nw, om.shape[1], int(k.shape[0]), len(temps)
    NQ = N ** 3
    kts = torch.as_tensor([_KB / _E * t for t in temps], device="cuda", dtype=torch.float64)
    f = 1.0 / (torch.exp((eps[:, :, None] - mu) / kts) + 1.0)            # [p][m][t]
    b = torch.where(live[:, :, None], 1.0 / torch.expm1(om.clamp(min=1e-30)[:, :, None] / kts), torch.zeros((), device="cuda", dtype=torch.float64))
    i = torch.arange(NQ, device="cuda")
    q1, q2, q3 = i % N, (i // N) % N, i // (N * N)
    g = torch.as_tensor(s.gw, device="cuda")                             # [re][rp][mu][i][j]
    gk = g.permute(0, 4, 1, 2, 3).reshape(s.re.shape[0] * nw, -1).contiguous()  # [(re, j)][(rp, mu, i)]
    re = torch.as_tensor(s.re, device="cuda").double()
    rp = np.mod(s.rp.astype(np.int64), N)
    ridx = torch.as_tensor(rp[:, 0] + N * (rp[:, 1] + N * rp[:, 2]), device="cuda")
    pref = 2.0 * math.pi / (_HBAR / _E) / NQ
    eta, cut = w.eta, 6.0 * w.eta
    dn = 1.0 / (math.sqrt(math.pi) * eta)
    out = torch.zeros(nt, ns, dtype=torch.float64, device="cuda")
    step = max(1, int(2e9 / (16.0 * NQ * nw * nm * 3)))
    ut = [[u[:, a, v].contiguous() for a in range(nm)] for v in range(nm)]
    for s0 in range(0, ns, step):
        kk, nn = k[s0:s0 + step], n[s0:s0 + step]
        nb = int(kk.shape[0])
        k3 = torch.stack([kk % N, (kk // N) % N, kk // (N * N)], 1).double()
        ph = torch.remainder(torch.round(k3 @ re.T), N) * (2.0 * math.pi / N)
        ph = torch.complex(torch.cos(ph), torch.sin(ph))                 # [b][re]
        vj = V[kk, :, nn]                                                # [b][j]
        X = ((ph[:, :, None] * vj[:, None, :]).reshape(nb, -1) @ gk).view(nb, s.rp.shape[0], nm * nw)
        box = torch.zeros(nb, nm * nw, NQ, dtype=torch.complex128, device="cuda")
        box.index_add_(2, ridx, X.transpose(1, 2).contiguous())
        G = torch.fft.ifftn(box.view(nb, nm * nw, N, N, N), dim=(2, 3, 4), norm="forward").view(nb, nm, nw, NQ)
        del box
        p = ((kk % N)[:, None] + q1) % N + N * ((((kk // N) % N)[:, None] + q2) % N + N * ((kk // (N * N))[:, None] + q3).remainder(N))
        es = eps[kk, nn][:, None]
        for m in range(nw):
            d = es - eps[p, m]
            vm = V[:, :, m].conj()
            W = torch.zeros(nb, nm, NQ, dtype=torch.complex128, device="cuda")
            for a in range(nw):
                W += vm[:, a][p][:, None, :] * G[:, :, a]
            acc = [torch.zeros(nb, NQ, dtype=torch.float64, device="cuda") for _ in range(nt)]
            fm = f[:, m]
            for v in range(nm):
                gg = torch.zeros(nb, NQ, dtype=torch.complex128, device="cuda")
                for a in range(nm):
                    gg += W[:, a] * ut[v][a]
                g2 = gg.real.square() + gg.imag.square()
                xp, xm = d + om[:, v], d - om[:, v]
                ok = live[:, v]
                dp = torch.where((xp.abs() <= cut) & ok, torch.exp(-(xp / eta) ** 2) * dn, torch.zeros_like(xp))
                dm = torch.where((xm.abs() <= cut) & ok, torch.exp(-(xm / eta) ** 2) * dn, torch.zeros_like(xm))
                for t in range(nt):
                    ft = fm[:, t][p]
                    acc[t] += g2 * ((b[:, v, t] + ft) * dp + (1.0 + b[:, v, t] - ft) * dm)
            for t in range(nt):
                out[t, s0:s0 + nb] += pref * acc[t].sum(1)
            if gamma_rows is not None:
                gamma_rows(s0, m, p, torch.stack(acc, 0) * pref)
    return out


def _exact_sigma(s_volume, nk, e, v, it, mu, temps, F=None, order=0):
    sig = torch.zeros(len(temps), 3, 3, dtype=torch.float64, device="cuda")
    for t, T in enumerate(temps):
        kt = _KB / _E * T
        f = 1.0 / (torch.exp((e - mu) / kt) + 1.0)
        wgt = f * (1.0 - f) / kt * (e - mu) ** order
        tau = torch.where(it[t] == 0.0, torch.zeros_like(it[t]), 1.0 / it[t])
        Ft = v * tau[:, None] if F is None else F[t]
        sig[t] = 2.0 * _E / (nk * s_volume * 1e-30) * ((v * wgt[:, None]).T @ Ft)
    return sig


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return None  # a chain of optimiser steps magnifies rounding: no one 64-bit result
    if kind == "transport":
        e, v, it, mu, temps = _state_arrays(case, seed)
        vol = abs(float(np.linalg.det(_system("toy_sc", 0).lattice)))
        m = [_exact_sigma(vol, 10 ** 6, e, v, it, mu, temps, order=o).cpu().numpy() for o in range(3)]
        see, kap = np.zeros_like(m[0]), np.zeros_like(m[0])
        for t, T in enumerate(temps):
            x = np.linalg.solve(m[0][t], m[1][t])
            see[t], kap[t] = -x / T, (m[2][t] - m[1][t] @ x) / T
        return dict(sigma=m[0], seebeck=see, kappa=kap)
    if kind == "predict":
        x, y = _samples(case, seed)
        x, y = x.double(), y.double()
        wt = torch.as_tensor(_weights(case, seed), device="cuda").double()
        h0 = (x - x.mean(0)) / x.std(0, unbiased=False)
        out = torch.empty(case["members"], case["samples"], case["n_out"], dtype=torch.float64, device="cuda")
        for m in range(case["members"]):
            h, at = h0, 0
            for layer, (fi, fo) in enumerate(((10, _WIDTH), (_WIDTH, _WIDTH), (_WIDTH, _WIDTH), (_WIDTH, case["n_out"]))):
                W = wt[m, at:at + fo * fi].view(fo, fi)
                at += fo * fi
                h = h @ W.T + wt[m, at:at + fo]
                at += fo
                if layer < 3:
                    h = h * torch.sigmoid(h)
            out[m] = h * y.std(0, unbiased=False) + y.mean(0)
        return dict(y=out)
    N = case["grid"]
    nw, nm, nre, nrp = _SHAPE[case["system"]]
    states = _DENSITY[case["system"]][0] * nw * N ** 3 * case.get("subset", 1.0)
    cost = states * N ** 3 * (nw * nm / 12.0) * (nw * nm * (1 + nm) / 48.0) ** 0.5
    if cost > 6e9 or N ** 3 * nw ** 2 > 1.2e7:
        return None
    w, variant, mu, lo, hi, temps = _conditions(case, seed)
    s = _system(case["system"], variant)
    tables = _exact_tables(s, N)
    k, n = _exact_states(case, seed, s, tables, w, lo, hi)
    energy, vel = tables[0][k, n], tables[2][k, n]
    if kind == "rates":
        it = _exact_rates(s, N, w, tables, k, n, mu, temps)
        sig = _exact_sigma(s.cell_volume, N ** 3, energy, vel, it, mu, temps)
        return dict(k=None, n=None, energy=energy, vel=vel, inv_tau=it, sigma=sig, counts=None)
    ns = int(k.shape[0])
    if ns > 14000:
        return None
    at = torch.full((N ** 3, nw), -1, dtype=torch.int64, device="cuda")
    at[k, n] = torch.arange(ns, device="cuda")
    A = torch.zeros(len(temps), ns, ns, dtype=torch.float64, device="cuda")

    def rows(s0, m, p, val):
        col = at[:, m][p]
        for r in range(p.shape[0]):
            keep = col[r] >= 0
            A[:, s0 + r, col[r][keep]] = val[:, r, keep]

    it = _exact_rates(s, N, w, tables, k, n, mu, temps, rows)
    F0 = vel[None] / it[:, :, None]
    F = F0.clone()
    sig = [_exact_sigma(s.cell_volume, N ** 3, energy, vel, it, mu, temps, F=F)]
    for _ in range(case["iterations"]):
        F = torch.stack([F0[t] + (A[t] @ F[t]) / it[t][:, None] for t in range(len(temps))])
        sig.append(_exact_sigma(s.cell_volume, N ** 3, energy, vel, it, mu, temps, F=F))
    return dict(k=None, n=None, inv_tau=it, sigma=torch.stack(sig), F=F, iterations=None, entries=None, bytes=None)
