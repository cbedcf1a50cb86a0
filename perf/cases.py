"""Performance cases of the Hermite N-body library: what its users have it do.

Every case is a dict of plain values; ``listed()`` names the fixed ones and
``draw(rng)`` gives one more of the same ranges.  ``prepare`` builds the
device state a user's program holds before the call, ``run`` makes the call
through the public binding (``paper_1104_2700_amd.hermite``), ``work`` counts
what the call cannot do without, and ``exact`` is the same result in plain
64-bit torch, without the library.

Kinds of case
-------------
force     ``Context.force_jerk``: acceleration, jerk and potential of an
          active block (or of every particle) of one system at the predicted
          positions; the caller keeps its output tensors.
ensemble  the same for an ensemble of independent clusters, all particles
          active, one call.
run       ``Context.run``: block steps of a system (or an ensemble) from its
          initialised state, restarted from a saved snapshot each pass.
step      ``Context.step`` called by the program itself, step by step.
energy    ``Context.energy``: the kinetic and potential energy that a run is
          checked with.

Sizes and settings are those of the repository's workloads: Plummer spheres
of 1024 to 65536 particles with eps = 4/N, clusters of 256 to 8192
particles, a Salpeter spectrum with 10 % binaries at 131072, eta = 0.02 with
the printed criterion, 2^-20 ticks, steps 2^-3 ... 2^-20.  Launch shapes and
the mixed-precision policy are the library's defaults.
"""
from __future__ import annotations

import math

import numpy as np
import torch

TICK_BITS = 20
ETA = 0.02
K_MIN, K_MAX = 3, 20
EPS_IMF = 1e-5


def listed():
    return [
        # The start of every run and every full-N evaluation of the 65536-body
        # sphere, in the reference precision.
        {"name": "force_fp64_n65536", "kind": "force", "n": 65536, "n_act": 65536,
         "precision": "fp64", "imf": False},
        # The same in the mixed precision: the headline sweep.
        {"name": "force_mixed_n65536", "kind": "force", "n": 65536, "n_act": 65536,
         "precision": "mixed", "imf": False},
        # A full evaluation of a mid-sized system whose size is no multiple of
        # anything.
        {"name": "force_fp64_n9973", "kind": "force", "n": 9973, "n_act": 9973,
         "precision": "fp64", "imf": False},
        # A large block of the 65536-body sphere: the coarse levels of a block
        # step, in the mixed precision.
        {"name": "block_mixed_n65536_a3001", "kind": "force", "n": 65536, "n_act": 3001,
         "precision": "mixed", "imf": False},
        # A block of the 131072-body system with a mass spectrum and binaries,
        # two-float sums.
        {"name": "block_mixed2f_imf_n131072_a1500", "kind": "force", "n": 131072,
         "n_act": 1500, "precision": "mixed2f", "imf": True},
        # The usual block of a 65536-body run: a few hundred particles.
        {"name": "block_fp64_n65536_a333", "kind": "force", "n": 65536, "n_act": 333,
         "precision": "fp64", "imf": False},
        # The smallest calls: a handful of particles of a small system.
        {"name": "block_fp64_n1024_a7", "kind": "force", "n": 1024, "n_act": 7,
         "precision": "fp64", "imf": False},
        # All particles of 256 clusters of 263 ... 8080 particles in one call
        # (the default mixed policy).
        {"name": "ensemble_mixed_c256", "kind": "ensemble", "clusters": 256, "n_min": 256,
         "n_max": 8192, "precision": "mixed"},
        # Integrating a small system: latency of a block step.
        {"name": "run_fp64_n1024", "kind": "run", "n": 1024, "clusters": 0, "steps": 256,
         "precision": "fp64"},
        # Integrating a mid-sized system.
        {"name": "run_fp64_n16384", "kind": "run", "n": 16384, "clusters": 0, "steps": 256,
         "precision": "fp64"},
        # Integrating an ensemble on one block timeline.
        {"name": "run_mixed_c64", "kind": "run", "n": 0, "clusters": 64, "n_min": 256,
         "n_max": 8192, "steps": 128, "precision": "mixed"},
        # The energy check of a run.
        {"name": "energy_n50021", "kind": "energy", "n": 50021},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["force", "block", "block", "ensemble", "run", "run", "run_ensemble",
                       "step", "energy"])
    if kind == "force":
        n = _log_int(rng, 700, 60000)
        return {"kind": "force", "n": n, "n_act": n, "imf": False,
                "precision": rng.choice(["fp64", "fp64", "mixed", "mixed2f", "mixed_sp"])}
    if kind == "block":
        imf = rng.random() < 0.25
        n = _log_int(rng, 1000, 30000 if imf else 65536)
        return {"kind": "force", "n": n, "n_act": _log_int(rng, 1, n // 2), "imf": imf,
                "precision": rng.choice(["fp64", "fp64", "mixed", "mixed2f"])}
    if kind == "ensemble":
        c = _log_int(rng, 3, 200)
        return {"kind": "ensemble", "clusters": c, "n_min": rng.randint(64, 600),
                "n_max": rng.randint(1500, 8192), "precision": rng.choice(["fp64", "mixed"])}
    if kind == "run":
        return {"kind": "run", "n": _log_int(rng, 300, 24000), "clusters": 0,
                "steps": rng.randint(64, 200), "precision": rng.choice(["fp64", "mixed"])}
    if kind == "run_ensemble":
        return {"kind": "run", "n": 0, "clusters": _log_int(rng, 4, 60),
                "n_min": rng.randint(100, 600), "n_max": rng.randint(1000, 6000),
                "steps": rng.randint(64, 128), "precision": rng.choice(["fp64", "mixed"])}
    if kind == "step":
        return {"kind": "step", "n": _log_int(rng, 500, 40000), "steps": rng.randint(16, 64),
                "precision": "fp64"}
    return {"kind": "energy", "n": _log_int(rng, 500, 60000)}


# ---- inputs ---------------------------------------------------------------

def _cluster_sizes(case):
    """Log-uniform sizes of an ensemble's clusters (fixed by the case)."""
    c = case["clusters"]
    lo, hi = math.log(case["n_min"]), math.log(case["n_max"])
    return [int(round(math.exp(lo + (hi - lo) * (k + 0.5) / c))) for k in range(c)]


def _system(case, seed):
    """(x, v, m, offsets or None, eps2 per system) as numpy arrays."""
    from paper_1104_2700_amd import inputs
    if case.get("clusters"):
        sizes = np.random.default_rng(seed).permutation(_cluster_sizes(case))
        parts = [inputs.plummer(int(k), 1000 * seed + c) for c, k in enumerate(sizes)]
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        x, v = (np.concatenate([p[q] for p in parts], axis=1) for q in (0, 1))
        return x, v, np.concatenate([p[2] for p in parts]), off, (4.0 / sizes) ** 2
    n = case["n"]
    if case.get("imf"):
        x, v, m = inputs.plummer_imf_binaries(n, seed)
        return x, v, m, None, EPS_IMF ** 2
    x, v, m = inputs.plummer(n, seed)
    return x, v, m, None, (4.0 / n) ** 2


def _active(case, seed):
    """The block's particle indices (ascending int32), or None for all."""
    from paper_1104_2700_amd import inputs
    if case["n_act"] == case["n"]:
        return None
    return inputs.random_active(case["n"], case["n_act"], seed + 1)


def prepare(case, seed):
    from paper_1104_2700_amd import hermite as H
    x, v, m, off, eps2 = _system(case, seed)
    st = {"case": case, "ctx": H.Context(0), "s": H.State(x, v, m, TICK_BITS),
          "eps2": 0.0 if off is not None else float(eps2),
          "cl": None if off is None else H.Clusters(off, eps2),
          "prec": H.PRECISIONS[case.get("precision", "fp64")]}
    s, kind = st["s"], case["kind"]
    if kind in ("force", "ensemble"):
        s.xp.copy_(s.x)
        s.vp.copy_(s.v)
        idx = _active(case, seed) if kind == "force" else None
        st["idx"] = None if idx is None else torch.from_numpy(idx).cuda()
        na = s.n if idx is None else idx.shape[0]
        st["out"] = [torch.empty(k, dtype=torch.float64, device="cuda")
                     for k in ((3, na), (3, na), (na,))]
    elif kind in ("run", "step"):
        st["params"] = H.dt_params(ETA, H.DT_PAPER, K_MIN, K_MAX)
        st["ctx"].initialize(s, st["eps2"], st["params"], st["prec"], clusters=st["cl"])
        st["start"] = s.clone()
    return st


def run(st):
    ctx, s, case = st["ctx"], st["s"], st["case"]
    kind = case["kind"]
    if kind in ("force", "ensemble"):
        acc, jerk, pot = st["out"]
        ctx.force_jerk(s, st["idx"], st["eps2"], st["prec"], acc=acc, jerk=jerk, pot=pot,
                       clusters=st["cl"])
        return {"acc": acc, "jerk": jerk, "pot": pot}
    if kind == "energy":
        return {"energy": ctx.energy(s, st["eps2"])}
    s.copy_from(st["start"])
    out = {}
    if kind == "run":
        out["steps"], out["interactions"] = ctx.run(
            s, st["eps2"], st["params"], 1 << TICK_BITS, st["prec"], use_graph=True,
            clusters=st["cl"], max_steps=case["steps"])
    else:
        for _ in range(case["steps"]):
            ctx.step(s, st["eps2"], st["params"], st["prec"], use_graph=True)
    for k in ("x", "v", "a", "j", "pot", "t", "dt"):
        out[k] = getattr(s, k)
    return out


# ---- what a pass cannot do without ------------------------------------------

# Per pair of particles that act on each other: differences 6, r^2 + eps^2 6,
# 1/sqrt 1, 1/s and its product 2, r.v 5, 3 (r.v)/s 2, v - b r 6; and for each
# of the two 1 + 1 for m/r and m/r^3, 1 potential, 6 acceleration, 6 jerk.
FLOPS_PAIR_SHARED, FLOPS_PAIR_SIDE = 28, 15


def work(case):
    kind = case["kind"]
    if kind in ("force", "ensemble"):
        sizes = _cluster_sizes(case) if kind == "ensemble" else [case["n"]]
        n = sum(sizes)
        if kind == "ensemble" or case["n_act"] == case["n"]:
            na = n
            flops = sum(0.5 * k * k * (FLOPS_PAIR_SHARED + 2 * FLOPS_PAIR_SIDE) for k in sizes)
        else:
            na = case["n_act"]
            flops = na * n * (FLOPS_PAIR_SHARED + FLOPS_PAIR_SIDE)
        return {"bytes": 56 * n + (4 + 56) * na, "flops": flops}
    if kind == "energy":
        n = case["n"]
        return {"bytes": 56 * n, "flops": 0.5 * n * n * (3 + 6 + 1 + 2 * 2)}
    # block steps: about 3 % of a system's particles per step (measured on
    # these spheres' first few hundred steps), each against its own system
    sizes = _cluster_sizes(case) if case.get("clusters") else [case["n"]]
    per_step = sum(max(1.0, 0.03 * k) * k for k in sizes)
    n = sum(sizes)
    return {"bytes": case["steps"] * (104 * n * 0.5 + 0.03 * n * 240),
            "flops": case["steps"] * per_step * (FLOPS_PAIR_SHARED + FLOPS_PAIR_SIDE)}


# ---- the same in plain 64-bit torch -------------------------------------------

def _pair_sums(x, v, m, rows, eps2, cells=1 << 25):
    """Sums over all j != i of one system for the rows i (int64 tensor)."""
    n = m.shape[0]
    acc, jerk, pot = [], [], []
    step = max(1, cells // n)
    for b in range(0, rows.shape[0], step):
        i = rows[b:b + step]
        r = [x[d][None, :] - x[d][i][:, None] for d in range(3)]
        w = [v[d][None, :] - v[d][i][:, None] for d in range(3)]
        s = r[0] * r[0] + r[1] * r[1] + r[2] * r[2] + eps2
        y = 1.0 / torch.sqrt(s)
        y[torch.arange(i.shape[0], device=y.device), i] = 0.0
        my = y * m
        my3 = my * y * y
        b3 = 3.0 * (r[0] * w[0] + r[1] * w[1] + r[2] * w[2]) / s
        b3 = torch.where(my3 == 0, torch.zeros_like(b3), b3)
        acc.append(torch.stack([(my3 * r[d]).sum(1) for d in range(3)]))
        jerk.append(torch.stack([(my3 * (w[d] - b3 * r[d])).sum(1) for d in range(3)]))
        pot.append(-my.sum(1))
    return torch.cat(acc, 1), torch.cat(jerk, 1), torch.cat(pot)


def _sums(x, v, m, rows, off, eps2):
    """_pair_sums over the systems [off[c], off[c+1]) of ascending rows."""
    if off is None:
        return _pair_sums(x, v, m, rows, eps2)
    parts = []
    cut = torch.searchsorted(rows, torch.as_tensor(off, device=rows.device)).tolist()
    for c in range(len(off) - 1):
        if cut[c] < cut[c + 1]:
            a, b = int(off[c]), int(off[c + 1])
            parts.append(_pair_sums(x[:, a:b], v[:, a:b], m[a:b], rows[cut[c]:cut[c + 1]] - a,
                                    float(eps2[c])))
    return tuple(torch.cat([p[q] for p in parts], -1) for q in range(3))


def _norm(u):
    return torch.sqrt((u * u).sum(0))


def _quantise(crit, k_old, T):
    """Steps in ticks: the largest 2^-k <= crit, at most twice the old one,
    dividing the block time T."""
    k = (1 - torch.frexp(crit).exponent.to(torch.int64)).clamp(K_MIN, K_MAX)
    if k_old is not None:
        k = torch.maximum(k, k_old - 1)
    if T:
        k = k.clamp(min=min(K_MAX, TICK_BITS - ((T & -T).bit_length() - 1)))
    return torch.ones_like(k) << (TICK_BITS - k)


def _integrate(x, v, m, off, eps2, steps):
    """Block steps from t = 0 (paper criterion), all in 64 bits."""
    n = m.shape[0]
    x, v = x.clone(), v.clone()
    a, j, pot = _sums(x, v, m, torch.arange(n, device=x.device), off, eps2)
    t = torch.zeros(n, dtype=torch.int64, device=x.device)
    dt = _quantise(ETA * _norm(a) / _norm(j), None, 0)
    tick = 2.0 ** -TICK_BITS
    for _ in range(steps):
        due = t + dt
        T = int(due.min())
        if T > 1 << TICK_BITS:
            break
        i = torch.nonzero(due == T).flatten()
        h = (T - t).to(torch.float64) * tick
        xp = x + h * (v + h * (a / 2 + h * j / 6))
        vp = v + h * (a + h * j / 2)
        a1, j1, p1 = _sums(xp, vp, m, i, off, eps2)
        h = dt[i].to(torch.float64) * tick
        da, a0, j0 = a[:, i] - a1, a[:, i], j[:, i]
        s0 = 2 * (-3 * da - (2 * j0 + j1) * h) / h ** 2
        c0 = 6 * (2 * da + (j0 + j1) * h) / h ** 3
        x[:, i] = xp[:, i] + s0 * h ** 4 / 24 + c0 * h ** 5 / 120
        v[:, i] = vp[:, i] + s0 * h ** 3 / 6 + c0 * h ** 4 / 24
        a[:, i], j[:, i], pot[i] = a1, j1, p1
        s1 = s0 + c0 * h
        A, J, S, C = _norm(a1), _norm(j1), _norm(s1), _norm(c0)
        crit = ETA * torch.sqrt((A * S + J * J) / (J * C + S * S))
        k_old = TICK_BITS - torch.log2(dt[i].to(torch.float64)).round().to(torch.int64)
        t[i] = T
        dt[i] = _quantise(crit, k_old, T)
    return x, v, a, j, pot


def exact(case, seed):
    x, v, m, off, eps2 = _system(case, seed)
    x, v, m = (torch.from_numpy(np.ascontiguousarray(u)).cuda() for u in (x, v, m))
    kind = case["kind"]
    if kind in ("force", "ensemble"):
        idx = _active(case, seed) if kind == "force" else None
        rows = (torch.arange(m.shape[0], device="cuda") if idx is None
                else torch.from_numpy(idx.astype(np.int64)).cuda())
        acc, jerk, pot = _sums(x, v, m, rows, off, eps2)
        return {"acc": acc, "jerk": jerk, "pot": pot}
    if kind == "energy":
        pot = _pair_sums(x, v, m, torch.arange(m.shape[0], device="cuda"), eps2)[2]
        kin = 0.5 * (m * (v * v).sum(0)).sum()
        return {"energy": torch.stack([kin, 0.5 * (m * pot).sum()])[None]}
    x, v, a, j, pot = _integrate(x, v, m, off, eps2, case["steps"])
    out = {"x": x, "v": v, "a": a, "j": j, "pot": pot, "t": None, "dt": None}
    if kind == "run":
        out["steps"] = out["interactions"] = None
    return out
