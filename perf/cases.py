"""Performance cases of the MLMC Dean--Kawasaki framework: the calls that its users make, from a
pilot batch that fills a corner of the GPU to the production batches of the finest levels, through
the entry points of ``paper_2311_08872_amd``.

``listed()`` names the cases, ``draw()`` gives further ones of the same ranges, ``prepare()`` makes
what a program holds before the call, ``run()`` is one call, ``work()`` what that call cannot do
without and ``exact()`` its values in 64 bits, written here in plain torch and numpy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import dk_workloads as W
import paper_2311_08872_amd as dk

DEV = "cuda:0"
OPS_PER_CELL = 121.0         # vector operations of one fine cell update (generator, transform, EM step)
BATCH_CAP = 8.0e10           # cell updates of the largest batch
EXACT_CAP = 9.0e9            # cell updates that the 64-bit reference takes in a few seconds


# ------------------------------------------------------------------------------------------
# The cases
# ------------------------------------------------------------------------------------------

def listed():
    return [
        # plain Monte Carlo of 16 x 16 paths, a pilot's 1000 samples: the smallest call, launch latency
        {"name": "mc_16_pilot", "kind": "batch", "problem": "config1", "N": 1e3, "level": 0, "coupled": False, "count": 1000},
        # the pilot batch (Algorithm 1's default 1000 samples) of a middle MLMC level
        {"name": "pair_32_pilot", "kind": "batch", "problem": "config2", "N": 1e4, "level": 2, "coupled": True, "count": 1000},
        # production batch of the finest resident level, where an MLMC run spends its time; 600 pairs
        # are not a whole number of rounds of the chip
        {"name": "pair_128_batch", "kind": "batch", "problem": "config2", "N": 1e4, "level": 4, "coupled": True, "count": 600},
        # low-density finest level: 256 x 256 pairs streamed through HBM, 29 observables
        {"name": "pair_256_stream", "kind": "batch", "problem": "config3", "N": 1e5, "level": 5, "coupled": True, "count": 40},
        # the paper's own setting (FP64 state), its finest grid
        {"name": "paper_128_f64", "kind": "batch", "problem": "paper_reg", "N": 2e9, "level": 5, "coupled": True, "count": 500},
        # the same setting with the Fourier coupling, its finest grid (108 x 108)
        {"name": "fourier_108_f64", "kind": "batch", "problem": "paper_fourier", "N": 2e9, "level": 3, "coupled": True,
         "count": 500},
        # Crank--Nicolson time stepping (b0 = 1/2) in the paper's setting, its finest grid
        {"name": "theta_64_f64", "kind": "batch", "problem": "paper_theta", "N": 2e9, "b0": 0.5, "level": 4, "coupled": True,
         "count": 1000},
        # the control variate's network over the coarse-only paths of 1000 pairs (4 each)
        {"name": "cnn_forward_64", "kind": "cnn_forward", "n": 64, "batch": 4000},
        # one training step's loss and gradient at the default batch
        {"name": "cnn_grad_64", "kind": "cnn_grad", "n": 64, "batch": 256},
        # the noise-free scheme on a batch of initial data, 64 steps in place
        {"name": "heat_256", "kind": "heat", "n": 256, "batch": 1000, "steps": 64, "mu": 0.1},
        # the discrete mean field that centres the observables of a streamed level
        {"name": "meanfield_512", "kind": "meanfield", "problem": "config5", "level": 5},
        # a whole Algorithm-1 run of the paper's setting from a fresh context (tables, mean fields, rounds)
        {"name": "estimate_paper", "kind": "estimate", "problem": "paper_reg", "N": 2e9, "eps": 10 ** -2.2},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["mc", "pair", "stream", "paper", "fourier", "theta", "cnn_forward", "cnn_grad", "heat", "meanfield",
                       "estimate"])
    if kind == "mc":
        c = {"kind": "batch", "problem": "config1", "N": round(_log(rng, 1e3, 1e5)), "n0": rng.choice([8, 16, 32]), "level": 0,
             "coupled": False, "flux": rng.choice([W.FLUX_CENTRAL, W.FLUX_STAGGERED])}
        return _counted(rng, c, 50, 20000)
    if kind == "pair":
        c = {"kind": "batch", "problem": "config2", "N": round(_log(rng, 1e3, 1e6)), "level": rng.randint(1, 4), "coupled": True,
             "flux": rng.choice([W.FLUX_CENTRAL, W.FLUX_CENTRAL, W.FLUX_STAGGERED]),
             "grid": rng.choice([W.GRID_VERTEX, W.GRID_VERTEX, W.GRID_CELL])}
        return _counted(rng, c, 50, 20000)
    if kind == "stream":
        if rng.random() < 0.5:
            c = {"kind": "batch", "problem": "config3", "N": round(_log(rng, 1e4, 1e7)), "level": 5,
                 "coupled": rng.random() < 0.7}
        else:
            c = {"kind": "batch", "problem": "config5", "N": 1e6, "level": rng.randint(4, 5), "coupled": rng.random() < 0.7}
        return _counted(rng, c, 4, 200)
    if kind == "paper":
        c = {"kind": "batch", "problem": rng.choice(["paper_reg", "paper_irreg"]), "N": rng.choice([2e5, 2e9]),
             "level": rng.randint(1, 5), "coupled": rng.random() < 0.7}
        return _counted(rng, c, 100, 8000)
    if kind == "fourier":
        c = {"kind": "batch", "problem": "paper_fourier", "N": rng.choice([2e5, 2e9]), "level": rng.randint(1, 3),
             "coupled": rng.random() < 0.75}
        return _counted(rng, c, 100, 4000)
    if kind == "theta":
        c = {"kind": "batch", "problem": "paper_theta", "N": rng.choice([2e5, 2e9]), "b0": rng.choice([0.5, 1.0]),
             "level": rng.randint(1, 4), "coupled": rng.random() < 0.75}
        return _counted(rng, c, 100, 4000)
    if kind in ("cnn_forward", "cnn_grad"):
        n = rng.choice([8, 16, 32, 64])
        most = 8192 if kind == "cnn_forward" else 512
        return {"kind": kind, "n": n, "batch": round(_log(rng, 32, most))}
    if kind == "heat":
        n = 4 * round(_log(rng, 32, 1024) / 4)
        return {"kind": "heat", "n": n, "batch": max(1, round(_log(rng, 2e6, 6e7) / n ** 2)), "steps": round(_log(rng, 1, 128)),
                "mu": rng.choice([0.05, 0.1, 0.25])}
    if kind == "meanfield":
        name, top = rng.choice([("config2", 4), ("config5", 5), ("paper_reg", 5)])
        return {"kind": "meanfield", "problem": name, "level": rng.randint(1, top), "N": rng.choice([1e4, 1e6])}
    return {"kind": "estimate", "problem": rng.choice(["paper_reg", "paper_irreg"]), "N": rng.choice([2e5, 2e9]),
            "eps": 10 ** rng.uniform(-2.5, -1.5)}


def _counted(rng, c, lo, hi):
    """c with a sample count, spread over its logarithm between lo and hi and within the largest batch."""
    p = _problem(c, 0)
    cap = min(hi, 0.6 * BATCH_CAP / (p.n(c["level"]) ** 2 * p.steps(c["level"])))
    c["count"] = max(1, round(_log(rng, min(lo, cap), cap)))
    return c


# ------------------------------------------------------------------------------------------
# The calls
# ------------------------------------------------------------------------------------------

def _problem(case, seed):
    name = case["problem"]
    if name == "config1":
        p = W.config1().with_(N=case["N"], n0=case.get("n0", 16))
    elif name == "config2":
        p = W.config2(case.get("N", 1e4)).with_(grid=case.get("grid", W.GRID_VERTEX))
    elif name == "config3":
        p = W.config3(case["N"])
    elif name == "config5":
        p = W.config5(case.get("N", 1e6))
    elif name == "paper_irreg":
        p = W.paper_irreg(case["N"])
    elif name == "paper_fourier":
        p = W.paper_fourier(case["N"])
    elif name == "paper_theta":
        p = W.paper_reg(case["N"]).with_(levels=5, b0=case["b0"])
    else:
        p = W.paper_reg(case["N"])
    return p.with_(seed=seed, flux=case.get("flux", W.FLUX_CENTRAL))


def _cnn_inputs(case, seed):
    """Network parameters (He initialisation), normalised coarse fields (unit-variance cells plus a smooth
    part) and standardised targets."""
    rng = np.random.default_rng(seed)
    params = np.zeros(5953, np.float32)
    for off, count, fan_in in ((0, 144, 9), (160, 2304, 144), (2480, 2304, 144), (4800, 1024, 16), (5888, 64, 64)):
        params[off:off + count] = rng.standard_normal(count) * math.sqrt(2.0 / fan_in)
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, b = case["n"], case["batch"]
    x = torch.randn((b, n, n), device=DEV, generator=g)
    x += torch.randn((b, 1, 1), device=DEV, generator=g) * torch.cos(
        2.0 * math.pi * torch.arange(n, device=DEV, dtype=torch.float32) / n)
    y = torch.randn((b,), device=DEV, generator=g)
    return params, x, y


def _heat_input(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return 1.0 + 0.5 * torch.rand((case["batch"], case["n"], case["n"]), device=DEV, generator=g)


def _meanfield_problem(case, seed):
    p = _problem(case, seed)
    rng = np.random.default_rng(seed)
    if p.rho0.kind == W.FIELD_EXPSIN2:
        f = p.rho0
        return p.with_(rho0=W.Field(f.kind, es_a=f.es_a, es_b=f.es_b, es_s=f.es_s, es_x0=float(rng.uniform(0, math.pi)),
                                    es_y0=float(rng.uniform(0, math.pi)), es_scale=f.es_scale))
    # the longest waves, which the observables see, beside shorter ones
    long_waves = [W.Mode(0.2, 1, 0, float(rng.uniform(0, math.pi))), W.Mode(0.2, 1, 1, float(rng.uniform(0, math.pi)))]
    return p.with_(rho0=W.Field(W.FIELD_MODES, 1.0, W.random_modes(6, seed) + long_waves))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "cnn_forward" or kind == "cnn_grad":
        params, x, y = _cnn_inputs(case, seed)
        return {"kind": kind, "ctx": dk.Context(0), "params": params, "x": x, "y": y}
    if kind == "heat":
        return {"kind": kind, "ctx": dk.Context(0), "rho": _heat_input(case, seed), "steps": case["steps"], "mu": case["mu"]}
    if kind == "meanfield":
        return {"kind": kind, "ctx": dk.Context(0), "problem": _meanfield_problem(case, seed), "level": case["level"]}
    if kind == "estimate":
        return {"kind": kind, "problem": _problem(case, seed), "eps": case["eps"]}
    return {"kind": kind, "ctx": dk.Context(0), "problem": _problem(case, seed), "level": case["level"],
            "coupled": case["coupled"], "count": case["count"]}


def _moments(ms):
    return np.array([[m.count] + list(m.sums) for m in ms], dtype=np.float64)


def run(state):
    kind = state["kind"]
    if kind == "batch":
        if state["coupled"]:
            ms, ps = dk.level_pair(state["problem"], state["level"], 0, state["count"], per_sample=True, ctx=state["ctx"])
        else:
            ms, ps = dk.mc_level(state["problem"], state["level"], 0, state["count"], per_sample=True, ctx=state["ctx"])
        return {"moments": _moments(ms), "per_sample": ps}
    if kind == "cnn_forward":
        return {"r": dk.cnn_forward(state["params"], state["x"], ctx=state["ctx"])}
    if kind == "cnn_grad":
        loss, grad = dk.cnn_loss_grad(state["params"], state["x"], state["y"], ctx=state["ctx"])
        return {"loss": loss, "grad": grad}
    if kind == "heat":
        dk.heat_steps(state["rho"], state["steps"], state["mu"], ctx=state["ctx"])
        return {"rho": state["rho"]}
    if kind == "meanfield":
        centre, rho = dk.meanfield(state["problem"], state["level"], want_field=True, ctx=state["ctx"])
        return {"centre": centre, "rho": rho}
    ctx = dk.Context(0)
    r = dk.estimate(state["problem"], state["eps"], ctx=ctx, level_moments=True)
    ctx.close()
    return {"estimate": r["estimate"], "var_est": r["var_est"], "bias_est": r["bias_est"], "L": r["L"], "M": r["M"],
            "Yhat": r["Yhat"], "Vhat": r["Vhat"], "moments": [_moments(m) for m in r["level_moments"][:r["L"] + 1]]}


# ------------------------------------------------------------------------------------------
# What a call cannot do without
# ------------------------------------------------------------------------------------------

def _batch_cells(p, level, coupled):
    per = p.n(level) ** 2 * p.steps(level)
    return per * (1.0 + p.ratio ** -4.0 if coupled else 1.0)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        p = _problem(case, 0)
        cells = case["count"] * _batch_cells(p, case["level"], case["coupled"])
        tables = p.n(case["level"]) ** 2 * 8.0 * (1 + len(p.obs)) * (1.25 if case["coupled"] else 1.0)
        return {"bytes": tables + case["count"] * len(p.obs) * 16.0, "flops": OPS_PER_CELL * cells}
    if kind == "cnn_forward" or kind == "cnn_grad":
        pix = float(case["batch"]) * case["n"] ** 2
        fwd = 2.0 * pix * (9 * 16 + 2 * 9 * 16 * 16)
        return {"bytes": 4.0 * pix + 4.0 * 5953, "flops": fwd if kind == "cnn_forward" else 3.0 * fwd}
    if kind == "heat":
        cells = float(case["batch"]) * case["n"] ** 2
        return {"bytes": 8.0 * cells, "flops": 7.0 * cells * case["steps"]}
    p = _problem(case, 0)
    if kind == "meanfield":
        n = p.n(case["level"])
        # into the eigenbasis of the separable stencil, one multiplier per mode, and back
        return {"bytes": 8.0 * n * n * (1 + len(p.obs)), "flops": 20.0 * n * n * math.log2(n)}
    # the pilot samples of the levels that the bias test visits
    top = 4 if case["eps"] < 10 ** -2.0 else 3
    return {"bytes": 16.0 * 1000 * (top + 1),
            "flops": OPS_PER_CELL * 1000 * sum(_batch_cells(p, l, l > 0) for l in range(top + 1))}


# ------------------------------------------------------------------------------------------
# 64-bit values
# ------------------------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        p = _problem(case, seed)
        if case["count"] * _batch_cells(p, case["level"], case["coupled"]) > EXACT_CAP or p.steps(case["level"]) > 1 << 14:
            return None
        return _exact_batch(p, case["level"], case["coupled"], case["count"])
    if kind == "cnn_forward":
        params, x, _ = _cnn_inputs(case, seed)
        return {"r": torch.cat([_network(torch.from_numpy(params).to(DEV).double(), xb) for xb in x.double().split(512)])}
    if kind == "cnn_grad":
        params, x, y = _cnn_inputs(case, seed)
        prm = torch.from_numpy(params).to(DEV).double().requires_grad_(True)
        loss = 0.0
        for xb, yb in zip(x.double().split(64), y.double().split(64)):
            part = ((_network(prm, xb) - yb) ** 2).sum() / case["batch"]
            part.backward()
            loss += float(part.detach())
        return {"loss": loss, "grad": prm.grad}
    if kind == "heat":
        n = case["n"]
        s = torch.sin(math.pi * torch.arange(n, device=DEV, dtype=torch.float64) / n) ** 2
        g = torch.exp(case["steps"] * torch.log1p(-2.0 * case["mu"] * (s[:, None] + s[None, :])))
        return {"rho": torch.cat([torch.fft.ifft2(torch.fft.fft2(f.double()) * g).real
                                  for f in _heat_input(case, seed).split(max(1, (1 << 25) // n ** 2))])}
    if kind == "meanfield":
        p = _meanfield_problem(case, seed)
        rho = _mean_field(p, case["level"])
        phi = _phis(p, case["level"])
        return {"centre": (p.h(case["level"]) ** 2 * (phi * rho).sum(dim=(1, 2))), "rho": rho}
    return None      # a whole run: its sample counts follow from its own estimates


def _field(p, f, n):
    """The analytic field f on the n x n grid, [y, x]."""
    c = (torch.arange(n, device=DEV, dtype=torch.float64) + p.offset) * (p.box / n)
    x, y = c[None, :].expand(n, n), c[:, None].expand(n, n)
    if f.kind == W.FIELD_EXPSIN2:
        return f.es_scale * (f.es_a + f.es_b * torch.exp(-(torch.sin(x - f.es_x0) ** 2 + torch.sin(y - f.es_y0) ** 2)
                                                         / (2.0 * f.es_s)))
    v = torch.full((n, n), float(f.c0), device=DEV, dtype=torch.float64)
    if f.kind == W.FIELD_BUMP:
        d2 = torch.zeros_like(v)
        for u, u0 in ((x, f.bump_cx), (y, f.bump_cy)):
            d = torch.remainder((u - u0).abs(), p.box)
            d2 = d2 + torch.minimum(d, p.box - d) ** 2
        return v + f.bump_amp * torch.exp(-d2 / (2.0 * f.bump_sigma ** 2))
    for m in f.modes:
        v = v + m.amp * torch.cos(2.0 * math.pi * (m.kx * x + m.ky * y) / p.box + m.phase)
    return v.clamp(min=0.0) + f.floor_add if f.kind == W.FIELD_CLIPPED else v


def _phis(p, level):
    return torch.stack([_field(p, o.phi, p.n(level)) for o in p.obs])


def _spectrum(p, n):
    s = torch.sin(math.pi * torch.arange(n, device=DEV, dtype=torch.float64) / n) ** 2
    return 2.0 * p.mu * (s[:, None] + s[None, :])


def _mean_field(p, level):
    n = p.n(level)
    lam = _spectrum(p, n)
    g = ((1.0 - (1.0 - p.b0) * lam) / (1.0 + p.b0 * lam)) ** p.steps(level) if p.b0 > 0 else \
        torch.exp(p.steps(level) * torch.log1p(-lam.clamp(max=1.0 - 1e-300))) if p.mu <= 0.25 else (1.0 - lam) ** p.steps(level)
    return torch.fft.ifft2(torch.fft.fft2(_field(p, p.rho0, n)) * g).real


def _exact_batch(p, level, coupled, count):
    out = torch.zeros((count, len(p.obs), 2), device=DEV, dtype=torch.float64)
    group = max(1, (1 << 24) // p.n(level) ** 2)
    for b in range(0, count, group):
        c = min(group, count - b)
        for slot, rho in enumerate(_paths(p, level, coupled, b, c)):
            l = level - slot
            phi, centre = _phis(p, l), _mean_field(p, l)
            for j, o in enumerate(p.obs):
                field = rho - centre if o.centre else rho
                v = p.h(l) ** 2 * (field * phi[j]).sum(dim=(1, 2)) * (math.sqrt(p.N) if o.scale_sqrtN else 1.0)
                out[b:b + c, j, slot] = v * v if o.psi == W.PSI_SQUARE else v
    ms = []
    for j in range(len(p.obs)):
        pf, pc = out[:, j, 0], out[:, j, 1]
        ms.append([float(count)] + [float(q.sum()) for v in (pf - pc, pf, pc) for q in (v, v * v)])
    return {"moments": np.array(ms), "per_sample": out}


def _paths(p, level, coupled, first, count):
    """Final fields of samples [first, first + count): [fine] or [fine, coarse]."""
    n, ratio = p.n(level), p.ratio
    m = ratio * ratio
    rho = _field(p, p.rho0, n).repeat(count, 1, 1)
    stepper = _stepper(p, n)
    if coupled:
        nc = p.n(level - 1)
        rhoc = _field(p, p.rho0, nc).repeat(count, 1, 1)
        coarse = _stepper(p, nc)
        K = _projection(n, nc) if ratio == 3 else None
        Z = 0.0
    # batches of steps whose noise is drawn at once: whole coarse steps, about 2^25 normals
    per = m * max(1, (1 << 24) // (n * n * count) // m)
    sig = math.sqrt(p.tau(level))
    for m0 in range(0, p.steps(level), per):
        k = min(per, p.steps(level) - m0)
        z = _normals(p.seed, W.TAG_MLMC if coupled else W.TAG_MC, level, n, first, count, m0, k)
        for j in range(k):
            rho = stepper(rho, z[j], sig)
            if not coupled:
                continue
            Z = Z + z[j]
            if (m0 + j) % m == m - 1:
                if K is None:
                    w = sum(Z[:, :, a::2, b::2] for a in (0, 1) for b in (0, 1))
                    rhoc = coarse(rhoc, w, 0.5 * sig)
                else:
                    # unit variance per coarse node: the coarse increment is h_c / h_f times sqrt(tau_f) / h-scale
                    rhoc = coarse(rhoc, torch.matmul(torch.matmul(K, Z), K.t().contiguous()), sig * ratio)
                Z = 0.0
    return [rho, rhoc] if coupled else [rho]


def _stepper(p, n):
    """One step of the scheme on fields [count, y, x] with unit normals z [direction, count, y, x] of size sigma."""
    h = p.box / n
    solve = 1.0 / (1.0 + p.b0 * _spectrum(p, n)) if p.b0 > 0 else None

    def step(rho, z, sigma):
        lap = rho.roll(1, 1) + rho.roll(-1, 1) + rho.roll(1, 2) + rho.roll(-1, 2) - 4.0 * rho
        if p.flux == W.FLUX_CENTRAL:
            root = rho.clamp(min=0.0).sqrt()
            f0, f1 = root * z[0], root * z[1]
            div = 0.5 * (f0.roll(-1, 2) - f0.roll(1, 2) + f1.roll(-1, 1) - f1.roll(1, 1))
        else:
            f0 = (0.5 * (rho + rho.roll(-1, 2))).clamp(min=0.0).sqrt() * z[0]
            f1 = (0.5 * (rho + rho.roll(-1, 1))).clamp(min=0.0).sqrt() * z[1]
            div = f0 - f0.roll(1, 2) + f1 - f1.roll(1, 1)
        d = 0.5 * p.mu * lap + (sigma / (math.sqrt(p.N) * h * h)) * div
        if solve is not None:
            d = torch.fft.ifft2(torch.fft.fft2(d) * solve).real
        return rho + d
    return step


def _projection(n, nc):
    """[nc][n] map of nodal noise onto the coarse frequencies, read at the coarse nodes."""
    d = 3.0 * torch.arange(nc, device=DEV, dtype=torch.float64)[:, None] - torch.arange(n, device=DEV, dtype=torch.float64)
    v = 1.0 + math.sqrt(2.0) * torch.cos(math.pi * nc * d / n)
    for k in range(1, nc // 2):
        v = v + 2.0 * torch.cos(2.0 * math.pi * k * d / n)
    return v / n


def _normals(seed, tag, level, n, first, count, m0, k):
    """The generator's normals of steps m0 .. m0 + k - 1: [step, direction, count, y, x] in 64 bits."""
    low = 0xFFFFFFFF
    pairs = n * n // 2
    a = torch.arange(pairs, device=DEV, dtype=torch.int64)
    step = torch.arange(m0, m0 + k, device=DEV, dtype=torch.int64)[:, None, None]
    s = torch.arange(first, first + count, device=DEV, dtype=torch.int64)[None, :, None]
    shape = (k, count, pairs)
    x, y = a.expand(shape), step.expand(shape)
    z, w = (s & low).expand(shape), ((tag << 24) | (level << 16) | ((s >> 32) & 0xFFFF)).expand(shape)
    k0, k1 = seed & low, (seed >> 32) & low
    for _ in range(10):
        p0, p1 = x * 0xD2511F53, z * 0xCD9E8D57
        x, y, z, w = ((p1 >> 32) & low) ^ y ^ k0, p1 & low, ((p0 >> 32) & low) ^ w ^ k1, p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    out = torch.empty((k, 2, count, n, n), device=DEV, dtype=torch.float64)
    grid = (k, count, n, n // 2)
    for c, (u, v) in enumerate(((x, y), (z, w))):
        z0, z1 = _box_muller(u, v)
        out[:, 0, :, :, c::2] = z0.view(grid)
        out[:, 1, :, :, c::2] = z1.view(grid)
    return out


def _box_muller(a, b):
    """The two normals of the words (a, b): Box and Muller's transform as the generator defines it, a fixed
    sequence of rounded binary32 operations (products of binary32 values are exact in 64 bits)."""
    f32, f64 = (lambda v: v.float()), (lambda v: v.double())

    def fma(u, v, c):
        return f32((f64(u) if torch.is_tensor(u) else u) * f64(v) + (f64(c) if torch.is_tensor(c) else c))

    def poly(coeffs, v):
        r = coeffs[0]
        for c in coeffs[1:]:
            r = fma(r, v, c)
        return r

    r32 = lambda v: float(np.float32(v))  # noqa: E731
    m, e = torch.frexp(f64(((a >> 9) << 1) | 1))
    fold = m > float.fromhex("0x1.6a09e6p-1")
    ne = f32(f64(e - 25 + fold.int()))
    xm = f32(torch.where(fold, m, 2.0 * m) - 1.0)
    g = [float.fromhex(v) for v in ("-0x1.0d33dap-3", "0x1.dbfb56p-3", "-0x1.e94d9cp-3", "0x1.fcc1c0p-3", "-0x1.231156p-2",
                                    "0x1.5554c0p-2", "-0x1.99a6e4p-2", "0x1.00002ap-1", "-0x1.555540p-1", "1.0", "-2.0")]
    lnm = xm * poly(g, xm)
    hi = ne * r32(float.fromhex("-0x1.62ep+0"))
    lo = fma(-2.0 * r32(0.69314718055994530942 - 0.693115234375), ne, lnm)
    R = f32(f64(hi + lo).sqrt())
    flip = (b >> 29) & 1
    j = ((b >> 7) & 0x7FFFFF) ^ (flip * 0x7FFFFF)
    c = float.fromhex("0x1.921fb6p-24")
    x = f32(f64(j) * (2.0 * c) + c)
    x2 = x * x
    sn = fma(x * x2, poly([r32(1.0 / 362880.0), r32(-1.0 / 5040.0), r32(1.0 / 120.0), r32(-1.0 / 6.0)], x2), x)
    cs = fma(x2, poly([r32(-1.0 / 3628800.0), r32(1.0 / 40320.0), r32(-1.0 / 720.0), r32(1.0 / 24.0), -0.5], x2), 1.0)
    q = b >> 30
    swap = (flip ^ (q & 1)) == 1
    co, si = torch.where(swap, sn, cs), torch.where(swap, cs, sn)
    co = torch.where((q == 1) | (q == 2), -co, co)
    si = torch.where(q >= 2, -si, si)
    return f64(R * co), f64(R * si)


def _network(prm, x):
    """The control variate's network on fields [batch, n, n]."""
    def conv(v, w, b):          # v [batch, n, n, in], w [out, in, 3, 3]
        s = b
        for i in range(9):
            s = s + v.roll((1 - i // 3, 1 - i % 3), (1, 2)) @ w[:, :, i // 3, i % 3].t().contiguous()
        return s.relu()
    v = conv(x[..., None], prm[:144].view(16, 1, 3, 3), prm[144:160])
    v = conv(v, prm[160:2464].view(16, 16, 3, 3), prm[2464:2480])
    v = conv(v, prm[2480:4784].view(16, 16, 3, 3), prm[4784:4800])
    h = (v.mean(dim=(1, 2)) @ prm[4800:5824].view(64, 16).t() + prm[5824:5888]).relu()
    return h @ prm[5888:5952] + prm[5952]
