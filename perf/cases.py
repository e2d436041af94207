"""The work that a user of this library has it do, as cases to measure.

Each case is one pass through the public Python binding
(``paper_1207_2367_amd``), from the smallest evaluation to a million-body one:

* ``force``: accelerations, jerks, snaps and potentials of an active set
  (``System.force``), the evaluation step of every block step and of any
  external integrator;
* ``noalloc``: the same from the caller's arrays (``force_noalloc``);
* ``init``: a new system, with its start-up evaluation (``System(...)``);
* ``energy``: the conservation check of a run (``System.energy``);
* ``snapshot``: the prediction of every particle to an output time and the
  checkpoint of the whole state (``System.predict``, ``System.get_state``);
* ``step``: resume from a checkpoint, advance by block steps, take the state
  (``System.set_state``, ``step``, ``get_state``), for one system or, with
  ``clusters``, for an ensemble of independent ones.

Inputs are Plummer spheres in Henon units (clusters of an ensemble: with a
spectrum of masses), softening 1e-4 or none, as in the paper's runs.
"""
import math

import numpy as np
import torch

from paper_1207_2367_amd import PREC_FP32PAIR, PREC_FP64, PREC_MIXED, System
from paper_1207_2367_amd.nbody import force_noalloc

PREC = {"mixed": PREC_MIXED, "fp64": PREC_FP64, "fp32pair": PREC_FP32PAIR}
B = 3.0 * math.pi / 16.0   # Plummer scale length in Henon units
F64 = torch.float64


def listed():
    return [
        # the smallest cluster of an ensemble, one particle due: pure latency
        {"name": "force_256x1", "kind": "force", "n": 256, "act": 1, "prec": "mixed", "eps": 1e-4},
        # a small block of the 65,536-body sphere (most block steps are of this size)
        {"name": "force_64k_x64", "kind": "force", "n": 65536, "act": 64, "prec": "mixed", "eps": 1e-4},
        # an odd-sized middle block without softening, on the FP64 path
        {"name": "force_100003x1237_fp64", "kind": "force", "n": 100003, "act": 1237, "prec": "fp64", "eps": 0.0},
        # a large block of a million-body sphere: nearly all of a long run's time
        {"name": "force_1m_x64k", "kind": "force", "n": 1048576, "act": 65536, "prec": "mixed", "eps": 1e-4},
        # evaluation inside a caller's own loop that may not allocate, fastest mode
        {"name": "noalloc_16k_x333_fp32", "kind": "noalloc", "n": 16384, "act": 333, "prec": "fp32pair", "eps": 1e-4},
        # start of a small run and of a benchmark-sized one
        {"name": "init_4k", "kind": "init", "n": 4096, "prec": "mixed", "eps": 1e-4},
        {"name": "init_64k", "kind": "init", "n": 65536, "prec": "mixed", "eps": 1e-4},
        # the energy check of a run of odd size
        {"name": "energy_100003", "kind": "energy", "n": 100003, "prec": "mixed", "eps": 1e-4},
        # output of a million-body run at a common time, and its checkpoint
        {"name": "snapshot_1m", "kind": "snapshot", "n": 1048573, "prec": "mixed", "eps": 1e-4},
        # block steps of the 1024-body sphere (small-block regime, one launch)
        {"name": "step_1k", "kind": "step", "n": 1024, "span": 0.0625, "prec": "mixed", "eps": 1e-4, "clusters": 1},
        # block steps of a middle-sized sphere (one block after another)
        {"name": "step_32k", "kind": "step", "n": 32768, "span": 0.015625, "prec": "mixed", "eps": 1e-4, "clusters": 1},
        # an ensemble of independent clusters of 256 to 4096 bodies
        {"name": "ensemble_48", "kind": "step", "n": 4096, "span": 0.03125, "prec": "mixed", "eps": 1e-4, "clusters": 48},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["force", "force", "force", "noalloc", "init", "energy", "snapshot", "step", "step"])
    case = {"kind": kind, "prec": rng.choice(["mixed", "mixed", "fp64", "fp32pair"]), "eps": rng.choice([1e-4, 1e-4, 0.0])}
    if kind == "force":
        case["n"] = _log(rng, 200, 1 << 20)
        case["act"] = _log(rng, 1, min(case["n"], (1 << 35) // case["n"]))
    elif kind == "noalloc":
        case["n"] = _log(rng, 200, 200000)
        case["act"] = _log(rng, 1, min(case["n"], 50000))
    elif kind == "init":
        case["n"] = _log(rng, 200, 60000)
    elif kind == "energy":
        case["n"] = _log(rng, 200, 200000)
    elif kind == "snapshot":
        case["n"] = _log(rng, 1000, 1000000)
    else:
        # runs are softened and not on the FP32-pair path (whose noise can
        # stop a run in a concentrated system)
        case["prec"], case["eps"] = rng.choice(["mixed", "fp64"]), 1e-4
        case["clusters"] = rng.choice([1, 1, rng.randint(3, 40)])
        case["n"] = _log(rng, 300, 24000 if case["clusters"] == 1 else 4000)
        case["span"] = 0.03125 if case["n"] <= 4096 else 0.0078125
    return case


# ------------------------------------------------------------------ inputs
def _plummer(n, g, dev, spectrum=False):
    """Positions by the inverse cumulative mass, speeds by the inverse
    cumulative of q^2 (1 - q^2)^(7/2), isotropic, centre-of-mass frame."""
    def unit(k):
        z = 2.0 * torch.rand(k, generator=g, dtype=F64, device=dev) - 1.0
        ph = 2.0 * math.pi * torch.rand(k, generator=g, dtype=F64, device=dev)
        s = torch.sqrt(1.0 - z * z)
        return torch.stack([s * torch.cos(ph), s * torch.sin(ph), z], 1)
    r = B / torch.sqrt((0.999 * torch.rand(n, generator=g, dtype=F64, device=dev)).clamp_min(1e-12) ** (-2.0 / 3.0) - 1.0)
    x = r[:, None] * unit(n)
    q = np.linspace(0.0, 1.0, 4097)
    c = np.cumsum(q * q * (1.0 - q * q) ** 3.5)
    c, q = (torch.as_tensor(t, dtype=F64, device=dev) for t in (c / c[-1], q))
    u = torch.rand(n, generator=g, dtype=F64, device=dev)
    k = torch.searchsorted(c, u).clamp(1, 4096)
    f = (u - c[k - 1]) / (c[k] - c[k - 1])
    v = (q[k - 1] + f * (q[k] - q[k - 1]))[:, None] * math.sqrt(2.0) * (r * r + B * B)[:, None] ** -0.25 * unit(n)
    m = torch.full((n,), 1.0 / n, dtype=F64, device=dev)
    if spectrum:   # dN/dm ~ m^-2.3 over one decade
        m = (1.0 - torch.rand(n, generator=g, dtype=F64, device=dev) * (1.0 - 10.0 ** -1.3)) ** (-1.0 / 1.3)
        m = m / m.sum()
    x = x - (m[:, None] * x).sum(0)
    v = v - (m[:, None] * v).sum(0)
    return m, x, v


def _sizes(case):
    """Clusters of an ensemble: sizes evenly spread in their logarithm from
    the largest down to a sixteenth of it (at least 2)."""
    k = case.get("clusters", 1)
    if k == 1:
        return [case["n"]]
    return [max(2, int(round(case["n"] * 16.0 ** (-i / (k - 1.0))))) for i in range(k)]


def _inputs(case, seed):
    """Everything a case starts from, from the seed alone."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 7919 + 13)
    sizes = _sizes(case)
    parts = [_plummer(k, g, dev, spectrum=len(sizes) > 1) for k in sizes]
    d = dict(zip("mxv", (torch.cat([p[q] for p in parts]) for q in range(3))))
    d["offsets"] = [0] + [int(o) for o in np.cumsum(sizes)]
    n = d["m"].shape[0]
    # the smooth model's acceleration for the sources
    d["a"] = -d["x"] / (((d["x"] ** 2).sum(1) + B * B) ** 1.5)[:, None]
    if "act" in case:
        d["idx"] = torch.randperm(n, generator=g, device=dev)[: case["act"]].sort().values.to(torch.int32)
    if case["kind"] == "snapshot":
        # derivatives of plausible size, block steps 2^-5 .. 2^-12, times at
        # multiples of the step below 1/4
        for q, key in enumerate(("jk", "sn", "cr")):
            d[key] = 4.0 ** (q + 1) * torch.randn((n, 3), generator=g, dtype=F64, device=dev)
        d["dt"] = 2.0 ** -torch.randint(5, 13, (n,), generator=g, device=dev).to(F64)
        d["t"] = torch.floor(0.25 / d["dt"] * torch.rand(n, generator=g, dtype=F64, device=dev)) * d["dt"]
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    kind, prec, eps = case["kind"], PREC[case["prec"]], case["eps"]
    st = {"case": case, "d": d}
    if kind in ("force", "energy", "snapshot"):
        st["s"] = System(d["m"], d["x"], d["v"], eps, precision=prec, skip_startup=True)
        st["s"].set_state(**{k: d[k] for k in ("a", "jk", "sn", "cr", "t", "dt") if k in d})
    elif kind == "step":
        st["s"] = System(d["m"], d["x"], d["v"], eps, precision=prec, offsets=d["offsets"])
        st["saved"] = st["s"].get_state()
    return st


def run(st):
    case, d = st["case"], st["d"]
    kind = case["kind"]
    if kind == "force":
        return st["s"].force(d["idx"])
    if kind == "noalloc":
        return force_noalloc(d["m"], d["x"], d["v"], d["a"], case["eps"], d["idx"], precision=PREC[case["prec"]])
    if kind == "init":
        s = System(d["m"], d["x"], d["v"], case["eps"], precision=PREC[case["prec"]])
        out = s.get_state()
        s.close()
        return out
    if kind == "energy":
        ekin, epot, L = st["s"].energy()
        return {"ekin": ekin, "epot": epot, "L": np.array(L)}
    if kind == "snapshot":
        return {"predicted": st["s"].predict(0.25), "state": st["s"].get_state()}
    st["s"].set_state(**st["saved"])
    stats = st["s"].step(case["span"])
    out = st["s"].get_state()
    out.update(block_steps=stats["block_steps"], active_total=stats["active_total"])
    return out


def work(case):
    """Operations by the count of 83 per pair of an evaluation (differences,
    r^2, 1/r, the terms of a, da, d2a and their sums; FMA = 2), 120 with the
    crackle, 45 without snap, 13 per pair of the energy; bytes: FP64 inputs
    and outputs once."""
    kind, n = case["kind"], sum(_sizes(case))
    if kind in ("force", "noalloc"):
        return {"bytes": 80.0 * n + 84.0 * case["act"], "flops": 83.0 * n * case["act"]}
    if kind == "init":
        return {"bytes": (56.0 + 160.0) * n, "flops": (45.0 + 120.0) * n * n}
    if kind == "energy":
        return {"bytes": 64.0 * n, "flops": 13.0 * 0.5 * n * n}
    if kind == "snapshot":
        return {"bytes": (152.0 + 72.0 + 2 * 160.0) * n, "flops": 102.0 * n}
    # about 110 (N / 1024)^0.3 steps per particle and unit of time
    pairs = sum(110.0 * (k / 1024.0) ** 0.3 * case["span"] * k * k for k in _sizes(case))
    return {"bytes": 2 * 160.0 * n, "flops": 83.0 * pairs}


# ------------------------------------------------------ reference, 64 bits
def _sums(d, idx, eps, acc, jrk=None, crackle=False):
    """a, da, d2a, (crackle,) potential of particles idx by direct sums."""
    m, x, v = d["m"], d["x"], d["v"]
    n, out = m.shape[0], []
    for k in torch.split(idx.long(), max(1, (1 << 25) // n)):
        def diff(q):
            return [q[None, :, c] - q[k, None, c] for c in range(3)]
        dx, dv, da = diff(x), diff(v), diff(acc)
        r2 = dx[0] ** 2 + dx[1] ** 2 + dx[2] ** 2 + eps * eps
        r2[torch.arange(k.shape[0], device=k.device), k] = math.inf   # no self term
        ri2 = 1.0 / r2
        w = m[None, :] * torch.sqrt(ri2)
        phi = -w.sum(1)
        w = w * ri2
        al = (dx[0] * dv[0] + dx[1] * dv[1] + dx[2] * dv[2]) * ri2
        be = (sum(dv[c] ** 2 for c in range(3)) + sum(dx[c] * da[c] for c in range(3))) * ri2 + al * al
        if crackle:
            dj = diff(jrk)
            ga = (3.0 * sum(dv[c] * da[c] for c in range(3)) + sum(dx[c] * dj[c] for c in range(3))) * ri2 + al * (3.0 * be - 4.0 * al * al)
        row = [[], [], [], []]
        for c in range(3):
            A = w * dx[c]
            J = w * dv[c] - 3.0 * al * A
            S = w * da[c] - 6.0 * al * J - 3.0 * be * A
            row[0].append(A.sum(1))
            row[1].append(J.sum(1))
            row[2].append(S.sum(1))
            if crackle:
                row[3].append((w * dj[c] - 9.0 * al * S - 9.0 * be * J - 3.0 * ga * A).sum(1))
        out.append([torch.stack(r, 1) for r in row if r] + [phi])
    return [torch.cat([o[q] for o in out]) for q in range(len(out[0]))]


def exact(case, seed):
    kind, eps = case["kind"], case["eps"]
    if kind == "step" or (kind in ("force", "noalloc") and case["n"] * case["act"] > 1 << 34):
        return None   # no plain 64-bit run of it within seconds
    d = _inputs(case, seed)
    n = d["m"].shape[0]
    if kind in ("force", "noalloc"):
        return tuple(_sums(d, d["idx"], eps, d["a"]))
    if kind == "init":
        every, zero = torch.arange(n, device=d["m"].device), torch.zeros_like(d["x"])
        a, j = _sums(d, every, eps, zero)[:2]
        s, c = _sums(d, every, eps, a, j, True)[2:4]
        na, nj, ns, nc = (torch.linalg.norm(q, dim=1) for q in (a, j, s, c))
        crit = 0.1 * torch.sqrt(na * ns + nj * nj) / torch.sqrt(nj * nc + ns * ns)
        dt = (2.0 ** torch.floor(torch.log2(crit))).clamp(max=1.0 / 16)
        return {"x": d["x"], "v": d["v"], "a": a, "jk": j, "sn": s, "cr": c, "t": torch.zeros_like(dt), "dt": dt}
    if kind == "energy":
        m, x, v = d["m"], d["x"], d["v"]
        every = torch.arange(n, device=m.device)
        phi = torch.cat([_phi(m, x, k, eps) for k in torch.split(every, max(1, (1 << 26) // n))])
        L = (m[:, None] * torch.linalg.cross(x, v)).sum(0)
        return {"ekin": float((0.5 * m * (v * v).sum(1)).sum()), "epot": float(0.5 * (m * phi).sum()), "L": L.cpu().numpy()}
    # snapshot: Taylor series to the output time, and the state as it is
    h = (0.25 - d["t"])[:, None]
    x, v, a, j, s, c = (d[k] for k in ("x", "v", "a", "jk", "sn", "cr"))
    p = (x + h * (v + h * (a / 2 + h * (j / 6 + h * (s / 24 + h * c / 120)))),
         v + h * (a + h * (j / 2 + h * (s / 6 + h * c / 24))),
         a + h * (j + h * (s / 2 + h * c / 6)))
    return {"predicted": p, "state": {"x": x, "v": v, "a": a, "jk": j, "sn": s, "cr": c, "t": d["t"], "dt": d["dt"]}}


def _phi(m, x, k, eps):
    r2 = sum((x[None, :, c] - x[k, None, c]) ** 2 for c in range(3)) + eps * eps
    r2[torch.arange(k.shape[0], device=k.device), k] = math.inf
    return -(m[None, :] / torch.sqrt(r2)).sum(1)
