"""Performance cases: the work a user has this library do, at the sizes of the
repository's own workloads.

Four kinds of work, each through the public Python entry points:

  steps   one subdomain advanced as the resolved-sample ramp does it: blocks of
          lattice steps, each followed by the FP64 reduction the steady-state
          test reads, and the density field read back at the end;
  ramp    the resumable drainage ramp of a packed sample, advanced by a number
          of lattice steps, with its results and the density field;
  batch   lbm_drain_batch on throats cut from a packing, the whole call;
  predict / train   the learned entry-pressure surrogate.

Every input follows from the seed.  Packings and the throats cut from them
are built once per process (host geometry), and the seed picks the throats,
perturbs the initial state or scales the pressures.
"""
import dataclasses
import functools
import math

import numpy as np
import torch

import synth
from paper_1906_04722_amd import lbm, surrogate
from synth import BC_PERIODIC, BC_RESERVOIR, BC_WALLS, Problem

BYTES_PER_UPDATE = 304    # 2 components x 19 FP32 populations, read and written
FLOPS_PER_UPDATE = 600
RHO_MINOR = 0.0609883
MEMBERS = 5
WIDTHS = (80, 256, 256, 256, 17)


def listed():
    return [
        # the smallest call: a 24^3 throat stepped a little, launch latency
        {"name": "throat_24", "kind": "steps", "box": "throat", "n": 24, "blocks": 1,
         "steps": 20, "tune": False},
        # the 40^3 four-sphere throat, as the parity tests and the smoke check run it
        {"name": "throat_40", "kind": "steps", "box": "throat", "n": 40, "blocks": 2,
         "steps": 100, "tune": False},
        # an odd box: ragged sides, walls, a periodic axis and baths, unequal tau
        {"name": "ragged_70x37x29", "kind": "steps", "box": "ragged", "nx": 70, "ny": 37,
         "nz": 29, "per_y": True, "tau_nw": 1.2, "blocks": 2, "steps": 100, "tune": False},
        # the 96^3 throat with lognormal radii, tuned as the benchmark does
        {"name": "throat_96", "kind": "steps", "box": "lognormal", "n": 96, "blocks": 4,
         "steps": 100, "tune": True},
        # the fully resolved 40-sphere sample with its outlet membrane, periodic
        # in x and y, checked every 200 steps as the full-sample ramp does
        {"name": "membrane_82", "kind": "steps", "box": "membrane", "res": 12.0, "blocks": 2,
         "steps": 200, "tune": True},
        # an all-fluid periodic box, memory bound
        {"name": "dense_256", "kind": "steps", "box": "dense", "n": 256, "blocks": 2,
         "steps": 100, "tune": True},
        # the packed sample (38 % fluid) on its drainage ramp, 400 lattice steps
        # a call as the benchmark's step; the largest case
        {"name": "sample_256", "kind": "ramp", "n": 256, "spheres": 125, "steps": 400,
         "tune": True},
        # batched drainage of small throats (the surrogate's and the hybrid's sizes)
        {"name": "batch_16_small", "kind": "batch", "throats": 16, "res": 12.0, "lo": 24,
         "hi": 64, "points": 4, "cap": 300},
        # batched drainage at the benchmark's resolution, box sides 48 to 128
        {"name": "batch_8_large", "kind": "batch", "throats": 8, "res": 32.0, "lo": 48,
         "hi": 128, "points": 4, "cap": 300},
        # the surrogate asked for the throats of one small packing
        {"name": "predict_64", "kind": "predict", "rows": 64},
        # and for a large set of descriptor rows
        {"name": "predict_100k", "kind": "predict", "rows": 100000},
        # training the ensemble on a drained set, batches of 64
        {"name": "train_456", "kind": "train", "rows": 456, "batch": 64, "epochs": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["throat", "throat", "lognormal", "ragged", "membrane", "dense", "ramp",
                       "batch", "predict", "train"])
    steps = 20 * _log_int(rng, 1, 10)
    if kind == "throat":
        return {"kind": "steps", "box": "throat", "n": _log_int(rng, 16, 64), "blocks":
                rng.randint(1, 3), "steps": steps, "tune": rng.random() < 0.5}
    if kind == "lognormal":
        return {"kind": "steps", "box": "lognormal", "n": _log_int(rng, 48, 128), "blocks":
                rng.randint(1, 3), "steps": steps, "tune": rng.random() < 0.7}
    if kind == "ragged":
        return {"kind": "steps", "box": "ragged", "nx": _log_int(rng, 17, 150),
                "ny": _log_int(rng, 17, 90), "nz": _log_int(rng, 17, 90),
                "per_y": rng.random() < 0.5, "tau_nw": rng.choice([1.0, 1.1, 1.2]),
                "blocks": rng.randint(1, 3), "steps": steps, "tune": rng.random() < 0.5}
    if kind == "membrane":
        return {"kind": "steps", "box": "membrane", "res": round(rng.uniform(5.0, 14.0), 2),
                "blocks": rng.randint(1, 2), "steps": steps, "tune": True}
    if kind == "dense":
        return {"kind": "steps", "box": "dense", "n": _log_int(rng, 24, 200), "blocks": 1,
                "steps": steps, "tune": True}
    if kind == "ramp":
        n = _log_int(rng, 64, 240)
        return {"kind": "ramp", "n": n, "spheres": 125, "steps": 100 * rng.randint(1, 4),
                "tune": True}
    if kind == "batch":
        large = rng.random() < 0.4
        return {"kind": "batch", "throats": rng.randint(2, 6 if large else 20),
                "res": 32.0 if large else 12.0, "lo": 48 if large else 24,
                "hi": 128 if large else 64, "points": rng.randint(2, 5),
                "cap": 100 * rng.randint(1, 3)}
    if kind == "predict":
        return {"kind": "predict", "rows": _log_int(rng, 1, 90000)}
    return {"kind": "train", "rows": _log_int(rng, 40, 900), "batch":
            rng.choice([16, 33, 64, 128]), "epochs": rng.randint(1, 4)}


# ---- inputs ------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _sample(n, spheres):
    return synth.packed_sample(n=n, n_spheres=spheres, seed=4)[0]


@functools.lru_cache(maxsize=None)
def _forty():
    return synth.dense_packing(40, seed=7)[:3]


@functools.lru_cache(maxsize=None)
def _throat_pool(res, lo, hi):
    probs, rins, _ = synth.packing_throats(n_throats=32, n_spheres=100, seed=3, res=res,
                                           side_range=(lo, hi), amp=0)
    return probs, rins


def _problem(case, seed):
    """The subdomain of a `steps` or `ramp` case."""
    if case["kind"] == "ramp":
        return _sample(case["n"], case["spheres"])
    box = case["box"]
    if box == "throat":
        if case["n"] == 40:
            return synth.c1_problem(seed=seed)
        return synth.small_throat_problem(n=case["n"], seed=seed)
    if box == "lognormal":
        p = synth.c2_problem(seed=seed, n=case["n"], mean_r=case["n"] / 3.0)
        return dataclasses.replace(p, probe=None)  # a seed can put it on a solid node
    rng = np.random.default_rng(seed)
    if box == "membrane":
        p = synth.membrane_sample(*_forty(), res=case["res"])[0]
        return dataclasses.replace(p, rho_in_nw=2.0 + 0.02 * (1.0 + rng.random()),
                                   z_front=p.z_front + int(rng.integers(0, 8)))
    if box == "dense":
        n = case["n"]
        return Problem(nx=n, ny=n, nz=n, bc=(BC_PERIODIC,) * 3, G_ads=(0.0, 0.0),
                       z_front=n // 2 - int(rng.integers(0, n // 8 + 1)),
                       rho_major=2.0 * (1.0 + 0.002 * rng.random()))
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    r = min(nx, ny, nz) / 4.5
    sph = np.array([[0.28 * nx, 0.38 * ny, 0.42 * nz, r],
                    [0.74 * nx, 0.68 * ny, 0.52 * nz, 0.85 * r],
                    [0.47 * nx, 0.82 * ny, 0.75 * nz, 0.55 * r]])
    sph[:, :3] += rng.uniform(-0.5, 0.5, (3, 3))
    rho0 = synth.layered_density(nx, ny, nz, nz // 5, 2.0, RHO_MINOR, seed=seed, amp=1e-3)
    return Problem(nx=nx, ny=ny, nz=nz, spheres=sph, tau=(1.0, case["tau_nw"]), rho_init=rho0,
                   bc=(BC_WALLS, BC_PERIODIC if case["per_y"] else BC_WALLS, BC_RESERVOIR),
                   rho_in_nw=2.03)


def _pressures(case, seed):
    scale = 0.9 + 0.2 * float(np.random.default_rng(seed).random())
    p = _sample(case["n"], case["spheres"])
    r_pore = 0.25 * float(np.mean(p.spheres[:, 3]))
    return scale * synth.pc_ramp(synth.GAMMA_LAPLACE, r_pore, 12)


RAMP = dict(tol=1e-6, check_every=100, max_steps=2000, bisect_rel=0.01)


def _throats(case, seed):
    probs, rins = _throat_pool(case["res"], case["lo"], case["hi"])
    rng = np.random.default_rng(seed)
    pick = rng.permutation(len(probs))[:case["throats"]]
    out = [dataclasses.replace(probs[i], rho_init=synth.layered_density(
        probs[i].nx, probs[i].ny, probs[i].nz, probs[i].z_front, probs[i].rho_major,
        probs[i].rho_minor, seed=seed + int(i), amp=1e-3)) for i in pick]
    pcs = np.array([synth.pc_ramp(synth.GAMMA_LAPLACE, rins[i], case["points"]) for i in pick])
    return out, pcs


def _features(rows, rng):
    """Rows like the descriptor's: 4 radii, 12 centre coordinates in mean
    radii, 64 block solid fractions."""
    return np.column_stack([np.exp(0.2 * rng.standard_normal((rows, 4))),
                            1.2 * rng.standard_normal((rows, 12)),
                            rng.beta(0.6, 0.4, (rows, 64))])


def _targets(F, rng):
    """p_c^e times the MS-P radius, then 16 falling saturations."""
    a = 0.19 * (1.0 + 0.1 * np.tanh(F[:, 0] - F[:, 1] + 0.3 * F[:, 4]))
    drop = np.cumsum(rng.uniform(0.0, 0.08, (F.shape[0], 16)), axis=1)
    return np.column_stack([a, 1.0 - drop * F[:, 16:17]])


def _weights(rng):
    out = []
    for _ in range(MEMBERS):
        parts = []
        for k, n in zip(WIDTHS[:-1], WIDTHS[1:]):
            a = math.sqrt(3.0 / k)
            parts += [rng.uniform(-a, a, n * k), 0.05 * rng.standard_normal(n)]
        out.append(np.concatenate(parts).astype(np.float32))
    return out


def _model_inputs(case, seed):
    rng = np.random.default_rng(seed)
    W = _weights(rng)
    F = _features(case["rows"], rng)
    if case["kind"] == "predict":
        S = _features(512, rng)
        stats = (S.mean(0), S.std(0), np.concatenate([[0.19], np.linspace(0.95, 0.4, 16)]),
                 np.concatenate([[0.02], np.full(16, 0.1)]))
        return W, F, stats
    T = _targets(F, rng)
    order = np.stack([np.stack([rng.permutation(case["rows"]) for _ in range(MEMBERS)])
                      for _ in range(case["epochs"])]).astype(np.int32)
    return W, F, T, order


def prepare(case, seed):
    if case["kind"] in ("steps", "ramp"):
        g = lbm.Throat(_problem(case, seed))
        if case["tune"]:
            g.autotune(5)
        if case["kind"] == "ramp":
            g.drain_begin(_pressures(case, seed), **RAMP)
        return case, g
    if case["kind"] == "batch":
        return (case,) + _throats(case, seed)
    m = surrogate.Surrogate(members=MEMBERS, seed=1)
    W, F, *rest = _model_inputs(case, seed)
    for z in range(MEMBERS):
        m.set_params(z, W[z])
    if case["kind"] == "predict":
        m.set_stats(*rest[0])
        return case, m, F
    return (case, m, F) + tuple(rest)


# ---- one pass ----------------------------------------------------------------

def run(state):
    case = state[0]
    if case["kind"] == "steps":
        g = state[1]
        S = np.zeros(case["blocks"])
        for b in range(case["blocks"]):
            g.step(case["steps"])
            mass, S[b] = g.reduce()
        return {"density": g.density(), "mass": mass, "S": S}
    if case["kind"] == "ramp":
        g = state[1]
        g.drain_advance(case["steps"])
        r = g.drain_get()
        return {"density": g.density(), "S": r["S"], "steps": r["steps"], "status": r["status"]}
    if case["kind"] == "batch":
        out, _ = lbm.drain_batch(state[1], state[2], tol=1e-6, check_every=100,
                                 max_steps=case["cap"], bisect_rel=0.1)
        res = {k: np.stack([np.asarray(o[k]) for o in out])
               for k in ("S", "steps", "status", "pce_lo", "pce_hi", "invaded_at", "n_bisect",
                         "total_steps")}
        return res
    m = state[1]
    if case["kind"] == "predict":
        mean, std = m.predict(state[2])
        return {"mean": mean, "std": std}
    hist = m.train(state[2], state[3], epochs=case["epochs"], batch=case["batch"], lr=1e-3,
                   order=state[4])
    return {"hist": hist, "weights": [m.get_params(z) for z in range(MEMBERS)]}


# ---- what one pass cannot do without -------------------------------------------

def work(case):
    if case["kind"] in ("steps", "ramp"):
        p = _problem(case, 0)
        n = case["steps"] * case.get("blocks", 1) * _fluid(_key(case))
        # the density field is written once more and handed to the host
        return {"bytes": BYTES_PER_UPDATE * n + 16 * p.n_nodes, "flops": FLOPS_PER_UPDATE * n}
    if case["kind"] == "batch":
        probs, _ = _throats(case, 0)
        # ramp points at their step cap; the bisection runs depend on the physics
        n = case["points"] * case["cap"] * sum(int((_classes(p) == 0).sum()) for p in probs)
        return {"bytes": BYTES_PER_UPDATE * n, "flops": FLOPS_PER_UPDATE * n}
    params = sum(k * n + n for k, n in zip(WIDTHS[:-1], WIDTHS[1:]))
    mul = sum(k * n for k, n in zip(WIDTHS[:-1], WIDTHS[1:]))
    rows = case["rows"]
    if case["kind"] == "predict":
        return {"bytes": 8 * rows * (80 + 34) + 4 * MEMBERS * params,
                "flops": 2 * mul * MEMBERS * rows}
    return {"bytes": case["epochs"] * -(-rows // case["batch"]) * 24 * MEMBERS * params,
            "flops": 6 * mul * MEMBERS * rows * case["epochs"]}


def _key(case):
    return tuple(sorted((k, v) for k, v in case.items() if k != "name"))


@functools.lru_cache(maxsize=None)
def _fluid(key):
    return int((_classes(_problem(dict(key), 0)) == 0).sum())


# ---- the same results in 64 bits, in plain numpy and torch -----------------------

E = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
              (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1),
              (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)])
OPP = [0] + [k + 1 if k % 2 else k - 1 for k in range(1, 19)]
WK = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)


def _classes(p):
    """Node classes [nz][ny][nx]: 0 fluid, 1 solid, 2 inlet bath, 3 outlet bath."""
    t = np.zeros((p.nz, p.ny, p.nx), dtype=np.uint8)
    side = (p.nx, p.ny, p.nz)
    for c in np.asarray(p.spheres, dtype=np.float64).reshape(-1, 4):
        lo = [max(0, int(math.floor(c[a] - c[3]))) for a in range(3)]
        hi = [min(side[a] - 1, int(math.ceil(c[a] + c[3]))) for a in range(3)]
        if any(h < l for l, h in zip(lo, hi)):
            continue
        x, y, z = [np.arange(l, h + 1) - c[a] for a, (l, h) in enumerate(zip(lo, hi))]
        d2 = (x * x)[None, None, :] + (y * y)[None, :, None]
        d2 = d2 + (z * z)[:, None, None]
        t[lo[2]:hi[2] + 1, lo[1]:hi[1] + 1, lo[0]:hi[0] + 1][d2 <= c[3] * c[3]] = 1
    if p.prism_ids is not None:
        A, B, C = [np.asarray(p.spheres, dtype=np.float64)[i] for i in p.prism_ids]
        x, y = np.arange(p.nx, dtype=np.float64)[None, :], np.arange(p.ny, dtype=np.float64)[:, None]

        def edge(P, Q, X, Y):
            return (Q[0] - P[0]) * (Y - P[1]) - (Q[1] - P[1]) * (X - P[0])
        s = 1.0 if edge(A, B, C[0], C[1]) > 0 else -1.0
        inside = (s * edge(A, B, x, y) >= 0) & (s * edge(B, C, x, y) >= 0) & \
            (s * edge(C, A, x, y) >= 0)
        t[:, ~inside] = 1
    if p.bc[2] == BC_RESERVOIR:
        t[0][t[0] == 0] = 2
        t[-1][t[-1] == 0] = 3
    return t


def _exact_steps(p, blocks, steps, rho_in):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    t = torch.from_numpy(_classes(p)).to(dev)
    live = (t != 1).reshape(-1).nonzero().reshape(-1)
    M = live.numel()
    number = torch.full((t.numel(),), -1, dtype=torch.int64, device=dev)
    number[live] = torch.arange(M, device=dev)
    z, y, x = live // (p.nx * p.ny), (live // p.nx) % p.ny, live % p.nx

    def neighbour(e):
        """Live index of x + e, -1 on solid nodes and beyond walls."""
        out = torch.ones(M, dtype=torch.bool, device=dev)
        c = []
        for v, d, n, b in zip((x, y, z), e, (p.nx, p.ny, p.nz), p.bc):
            w = v + int(d)
            if b == BC_PERIODIC:
                w = w % n
            else:
                out &= (w >= 0) & (w < n)
                w = w.clamp(0, n - 1)
            c.append(w)
        return torch.where(out, number[(c[2] * p.ny + c[1]) * p.nx + c[0]], -1)

    nb = torch.stack([neighbour(E[k]) for k in range(19)])
    self_ = torch.arange(M, device=dev)
    pull = torch.stack([torch.where(nb[OPP[k]] >= 0, k * M + nb[OPP[k]], OPP[k] * M + self_)
                        for k in range(19)])
    e = torch.tensor(E, dtype=torch.float64, device=dev)
    wk = torch.tensor(WK, dtype=torch.float64, device=dev)
    A = torch.zeros(3, M, dtype=torch.float64, device=dev)
    for k in range(1, 19):
        A += (wk[k] * e[k])[:, None] * (nb[k] < 0)
    cls = t.reshape(-1)[live]
    fluid = cls == 0
    bath = {2: (p.rho_minor, rho_in), 3: (p.rho_out_w, p.rho_minor)}
    first = p.rho_init
    rho = []
    for c in range(2):
        if first is not None:
            r = torch.from_numpy(np.asarray(first[c], dtype=np.float64).reshape(-1)).to(dev)[live]
        else:
            nw = ((z <= p.z_front) == (c == 1)).double()
            r = nw * p.rho_major + (1.0 - nw) * p.rho_minor
        for b, v in bath.items():
            r = torch.where(cls == b, v[c], r)
        rho.append(r)
    f = [wk[:, None] * r for r in rho]
    phib = (p.rho_major - p.rho_minor) / (p.rho_major + p.rho_minor)

    def densities():
        out = []
        for c in range(2):
            r = f[c].sum(0)
            for b, v in bath.items():
                r = torch.where(cls == b, v[c], r)
            out.append(r)
        return out

    def reduced():
        a, b = [r[fluid] for r in densities()]
        return [float(a.sum()), float(b.sum())], \
            float((((a - b) / (a + b) + phib) / (2 * phib)).mean())

    S = []
    for _ in range(blocks):
        for _ in range(steps):
            rho = densities()
            pad = [torch.cat([r, r.new_zeros(1)]) for r in rho]  # index -1: no density
            force = []
            for c in range(2):
                s = torch.zeros(3, M, dtype=torch.float64, device=dev)
                for k in range(1, 19):
                    v = wk[k] * pad[1 - c][nb[k]]
                    for a in range(3):
                        if E[k][a]:
                            s[a] += int(E[k][a]) * v
                force.append(-p.G * rho[c] * s - p.G_ads[c] * rho[c] * A)
            mom = [e.T @ f[c] for c in range(2)]
            up = (mom[0] / p.tau[0] + mom[1] / p.tau[1]) / (rho[0] / p.tau[0] + rho[1] / p.tau[1])
            for c in range(2):
                u = up + p.tau[c] * force[c] / rho[c]
                eu = e @ u
                eq = wk[:, None] * rho[c] * (1 + 3 * eu + 4.5 * eu * eu - 1.5 * (u * u).sum(0))
                post = f[c] - (f[c] - eq) / p.tau[c]
                for b, v in bath.items():
                    at = cls == b
                    if bool(at.any()):
                        post = torch.where(at, wk[:, None] * v[c], post)
                f[c] = post.reshape(-1)[pull]
        mass, s = reduced()
        S.append(s)
    rho = densities()
    field = torch.zeros(2, t.numel(), dtype=torch.float64, device=dev)
    for c in range(2):
        field[c, live] = rho[c]
    return field.reshape(2, p.nz, p.ny, p.nx).cpu().numpy(), np.array(mass), np.array(S)


def _silu(z):
    return z / (1.0 + torch.exp(-z))


def _layers(w):
    out, o = [], 0
    for k, n in zip(WIDTHS[:-1], WIDTHS[1:]):
        out.append((w[:, o:o + n * k].reshape(-1, n, k), w[:, o + n * k:o + n * k + n]))
        o += n * k + n
    return out


def _forward(w, x):
    for i, (W, b) in enumerate(_layers(w)):
        x = torch.bmm(x, W.transpose(1, 2).contiguous()) + b[:, None, :]
        x = _silu(x) if i < 3 else x
    return x


def _exact_predict(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    W, F, (xm, xs, tm, ts) = _model_inputs(case, seed)
    w = torch.from_numpy(np.stack(W).astype(np.float64)).to(dev)
    x = torch.from_numpy((F - xm) / xs).to(dev)
    y = _forward(w, x.expand(MEMBERS, -1, -1).contiguous()).cpu().numpy() * ts + tm
    return {"mean": y.mean(0), "std": y.std(0)}


def _exact_train(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    W, F, T, order = _model_inputs(case, seed)
    w = torch.from_numpy(np.stack(W).astype(np.float64)).to(dev).requires_grad_(True)
    data = []
    for a in (F, T):
        sd = a.std(0)
        data.append(torch.from_numpy((a - a.mean(0)) / np.where(sd < 1e-12, 1.0, sd)).to(dev))
    m, v = torch.zeros_like(w), torch.zeros_like(w)
    per = -(-case["rows"] // case["batch"])
    total, hist = case["epochs"] * per, []
    for ep in range(case["epochs"]):
        losses = []
        for st in range(per):
            idx = torch.from_numpy(order[ep][:, st * case["batch"]:(st + 1) * case["batch"]]
                                   .astype(np.int64)).to(dev)
            loss = ((_forward(w, data[0][idx]) - data[1][idx]) ** 2).mean((1, 2))
            g, = torch.autograd.grad(loss.sum(), w)
            losses.append(loss.detach())
            i = ep * per + st + 1
            lr = 1e-3 * 0.5 * (1.0 + math.cos(math.pi * (i - 1) / total))
            with torch.no_grad():
                m = 0.9 * m + 0.1 * g
                v = 0.999 * v + 0.001 * g * g
                w -= lr * (m / (1 - 0.9 ** i)) / (torch.sqrt(v / (1 - 0.999 ** i)) + 1e-8)
        hist.append(float(torch.stack(losses).mean()))
    out = w.detach().cpu().numpy()
    return {"hist": np.array(hist), "weights": [out[z] for z in range(MEMBERS)]}


def exact(case, seed):
    if case["kind"] == "steps":
        p = _problem(case, seed)
        field, mass, S = _exact_steps(p, case["blocks"], case["steps"], p.rho_in_nw)
        return {"density": field, "mass": mass, "S": S}
    if case["kind"] == "ramp":
        p = _problem(case, seed)
        rho_in = p.rho_out_w + _pressures(case, seed)[0] / ((1.0 + p.G * p.rho_minor) / 3.0)
        field, _, _ = _exact_steps(p, 1, case["steps"], rho_in)
        return {"density": field, "S": None, "steps": None, "status": None}
    if case["kind"] == "predict":
        return _exact_predict(case, seed)
    if case["kind"] == "train":
        return _exact_train(case, seed)
    return None  # a batch's ramp decisions: hundreds of steps of every throat one by one
