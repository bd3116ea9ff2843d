"""The engine's work as its users have it done, case by case.

Every case goes through the public surface (``Plan``, ``ContinuousTime``,
``Coined``, ``Staggered``, ``evolve_many``, ``Batch``) with sizes from the
benchmark workloads, the serving stream and the tests, or generic ones:

cycle      a coined walk on a small cycle with its readout (the paper's
           Sec. 3.2 example size): one call of a few microseconds, latency
small      a group of small jobs of mixed kinds in one launch, as the serving
           loop sends them
grid       CTQW on a periodic grid, Taylor order given, one evolve and readout
sparse     CTQW on a sparse random graph through ContinuousTime.simulate, the
           states at a range of steps, order by the truncation rule
regular    CTQW search on a large random-looking regular graph
batch      ragged CTQW searches on regular graphs in one Batch, run to the end
hypercube  coined Grover search on a hypercube
gridwalk   coined Grover search on a grid (the serving stream's other family)
irregular  coined Grover walk on a sparse random graph (general CSR path)
lattice    persistent shift with the Fourier coin on a grid
squares    staggered search on the square lattice
dense      CTQW search on the complete graph, several walks sharing a dense H

States start random or uniform as such walks do; one pass advances them in
place, and norms are preserved, so passes can follow each other.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2406_08186_amd import inputs as I
from paper_2406_08186_amd.walk import Batch, ContinuousTime, Plan, Staggered, evolve_many


def listed():
    return [
        # the 64-cycle Hadamard walk: 100 steps, complex128, probabilities
        dict(name="cycle_64_c128", kind="cycle", n=64, coin="hadamard", steps=100, dtype="c128"),
        # a serving group of small jobs (cycles, grids, random graphs, squares)
        dict(name="small_48_c64", kind="small", count=48, nmax=1200, steps=100, dtype="c64"),
        # the 1024^2 grid CTQW, Taylor order 20 at dt 0.1
        dict(name="grid_1024_c64", kind="grid", l1=1024, l2=1024, K=20, dt=0.1, steps=100, marks=0, dtype="c64"),
        # simulate(range) on a sparse random graph, complex128, five states handed back
        dict(name="sparse_150001_c128", kind="sparse", n=150001, deg=10.0, dt=1.0, every=20, count=5, dtype="c128"),
        # a search on a large 6-regular graph, order by the rule at 1e-8
        dict(name="regular_1000000_c64", kind="regular", n=1000000, d=6, steps=40, dtype="c64"),
        # a batch of searches, N log-uniform in [1e3, 2e5], d in 3..8
        dict(name="batch_192_c64", kind="batch", count=192, nmin=1000, nmax=200000, steps=6, dtype="c64"),
        # hypercube search at the serving stream's largest size
        dict(name="hypercube_18_c64", kind="hypercube", dim=18, steps=200, dtype="c64"),
        # grid search of about 2e6 arcs, odd sides
        dict(name="gridwalk_707x709_c128", kind="gridwalk", l1=707, l2=709, steps=150, dtype="c128"),
        # Grover walk on an arbitrary sparse graph with a marked vertex
        dict(name="irregular_120000_c64", kind="irregular", n=120000, deg=9.0, steps=60, dtype="c64"),
        # Fourier coin, persistent shift, on a large grid
        dict(name="lattice_1024_c64", kind="lattice", l1=1024, l2=1024, steps=50, dtype="c64"),
        # staggered search on 2 x 2 squares
        dict(name="squares_768x1100_c128", kind="squares", l1=768, l2=1100, steps=60, dtype="c128"),
        # 32 searches sharing the dense H of a complete graph
        dict(name="dense_2500x32_c128", kind="dense", n=2500, columns=32, K=24, dt=0.65, steps=20, dtype="c128"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice([c["kind"] for c in listed()])
    dtype = rng.choice(["c64", "c128"])
    if kind == "cycle":
        return dict(kind=kind, n=_log(rng, 5, 1500), coin=rng.choice(["hadamard", "grover"]),
                    steps=rng.randint(1, 100), dtype=dtype)
    if kind == "small":
        return dict(kind=kind, count=rng.randint(2, 48), nmax=_log(rng, 40, 1200), steps=rng.randint(5, 100),
                    dtype=dtype)
    if kind == "grid":
        return dict(kind=kind, l1=_log(rng, 60, 1024), l2=_log(rng, 64, 1024), K=rng.randint(6, 24),
                    dt=rng.uniform(0.05, 0.8), steps=rng.randint(1, 100), marks=rng.randint(0, 3), dtype=dtype)
    if kind == "sparse":
        return dict(kind=kind, n=_log(rng, 3000, 150001), deg=rng.uniform(4.0, 14.0), dt=rng.uniform(0.4, 1.0),
                    every=_log(rng, 1, 20), count=rng.randint(2, 5), dtype=dtype)
    if kind == "regular":
        return dict(kind=kind, n=2 * _log(rng, 4000, 400000), d=rng.randint(3, 8), steps=rng.randint(2, 40),
                    dtype=dtype)
    if kind == "batch":
        return dict(kind=kind, count=_log(rng, 4, 190), nmin=1000, nmax=_log(rng, 5000, 150000),
                    steps=rng.randint(2, 6), dtype=dtype)
    if kind == "hypercube":
        return dict(kind=kind, dim=rng.randint(12, 17), steps=rng.randint(5, 200), dtype=dtype)
    if kind in ("gridwalk", "lattice"):
        return dict(kind=kind, l1=_log(rng, 60, 700), l2=_log(rng, 60, 700), steps=rng.randint(5, 150 if kind == "gridwalk" else 50),
                    dtype=dtype)
    if kind == "irregular":
        return dict(kind=kind, n=_log(rng, 3000, 110000), deg=rng.uniform(4.0, 9.0), steps=rng.randint(5, 60),
                    dtype=dtype)
    if kind == "squares":
        return dict(kind=kind, l1=2 * _log(rng, 60, 380), l2=2 * _log(rng, 60, 500), steps=rng.randint(5, 60),
                    dtype=dtype)
    return dict(kind=kind, n=_log(rng, 250, 2000), columns=rng.choice([1, 2, 5, 8, 16, 24, 32]), K=24,
                dt=rng.uniform(0.1, 0.65), steps=rng.randint(2, 20), dtype=dtype)


# ---- inputs ------------------------------------------------------------------

def _regular(n, d, seed):
    """A d-regular graph whose neighbours lie anywhere: a circulant with random
    offsets, its vertices relabelled by a random permutation (rows sorted).
    n even when d is odd."""
    rng = np.random.default_rng(seed)
    offs = rng.choice(np.arange(1, (n - 1) // 2 + 1), size=d // 2, replace=False).tolist()
    shifts = [s for o in offs for s in (o, n - o)] + ([n // 2] if d % 2 else [])
    perm = rng.permutation(n).astype(np.int32)
    nb = np.empty((n, d), dtype=np.int32)
    for j, s in enumerate(shifts):
        nb[perm, j] = np.roll(perm, -s)
    nb.sort(axis=1)
    return I.Graph(n, np.arange(0, n * d + 1, d, dtype=np.int64), nb.reshape(-1), f"regular{n}d{d}")


def _sparse_graph(n, deg, seed):
    """A random graph of n vertices and round(n deg / 2) edges: G(n, p) given its edge count."""
    rng, m = np.random.default_rng([seed, 3]), int(round(n * deg / 2))
    keys = np.empty(0, dtype=np.int64)
    while keys.size < m:
        a, b = rng.integers(0, n, size=(2, m - keys.size + 64))
        ok = a != b
        keys = np.unique(np.concatenate([keys, np.minimum(a, b)[ok] * n + np.maximum(a, b)[ok]]))
    keys = rng.choice(keys, size=m, replace=False)
    return I.from_edges(n, np.stack([keys // n, keys % n], 1), f"sparse{n}")


def _random(m, seed):
    rng = np.random.default_rng(seed)
    z = rng.standard_normal(2 * m).view(np.complex128)
    return z / np.linalg.norm(z)


def _uniform(m):
    return np.full(m, 1.0 / math.sqrt(m), dtype=np.complex128)


def _search(n, d):
    """Step length and horizon of a search on a d-regular graph: t = 2 sqrt(n) with
    gamma = 1/d, so ||H|| <= 2 and rho = dt ||H|| <= 1."""
    t = 2.0 * math.sqrt(n)
    steps = math.ceil(2.0 * t)
    return t / steps, steps


def _small_walks(case, seed):
    """(kind, graph, parameters, initial state, steps) of each job of a small group."""
    rng, size = np.random.default_rng([seed, 17]), np.random.default_rng([case["count"], case["nmax"]])
    out = []
    for i in range(case["count"]):
        s = int(rng.integers(1 << 30))
        n = int(round(math.exp(size.uniform(math.log(24), math.log(case["nmax"])))))
        steps = int(size.integers(max(1, case["steps"] // 2), case["steps"] + 1))
        mark = [int(rng.integers(16))]
        what = i % 5
        if what == 0:
            g = I.cycle(min(n, 600))
            out.append(("coined", g, dict(coin="hadamard"), _random(g.n_arcs, s), steps))
        elif what == 1:
            a = max(4, int(math.sqrt(min(n, 900))))
            g = I.torus(a, a + 1)
            out.append(("coined", g, dict(marked=mark), _uniform(g.n_arcs), steps))
        elif what == 2:
            g = I.erdos_renyi(n, min(0.5, 6.0 / n), s)
            h = 0.2 * int(np.diff(g.row_ptr).max()) + 1.0
            out.append(("ctqw", g, dict(gamma=0.2, dt=1.0 / h, trunc_tol=1e-10, horizon_steps=100, marked=mark),
                        _uniform(g.n), steps))
        elif what == 3:
            a = max(4, int(math.sqrt(n)))
            g = I.torus(a, a)
            out.append(("ctqw", g, dict(gamma=0.25, dt=0.1, taylor_order=12), _random(g.n, s), steps))
        else:
            a = max(4, int(math.sqrt(n)) // 2 * 2)
            g, tess = I.stag_lattice(a, a)
            out.append(("staggered", g, dict(tessellations=tess, marked=mark), _uniform(g.n), steps))
    return out


def _batch_walks(case, seed):
    rng, size = np.random.default_rng([seed, 29]), np.random.default_rng([case["count"], case["nmax"]])
    out = []
    for _ in range(case["count"]):
        n = int(round(math.exp(size.uniform(math.log(case["nmin"]), math.log(case["nmax"])))))
        d = int(size.integers(3, 9))
        n += (n * d) % 2
        dt, horizon = _search(n, d)
        out.append((_regular(n, d, int(rng.integers(1 << 30))), d, dt, horizon, int(rng.integers(n))))
    return out


def _walk(case, seed):
    """(walk kind, graph, plan parameters, initial state, steps) of a single-walk case."""
    k, dtype = case["kind"], case["dtype"]
    rng = np.random.default_rng([seed, 5])
    if k == "cycle":
        g = I.cycle(case["n"])
        psi = np.zeros(g.n_arcs, dtype=np.complex128)
        v, ph = int(rng.integers(g.n)), rng.uniform(0, 2 * math.pi)
        psi[2 * v], psi[2 * v + 1] = 1 / math.sqrt(2), np.exp(1j * ph) / math.sqrt(2)
        return "coined", g, dict(coin=case["coin"]), psi, case["steps"]
    if k == "grid":
        g = I.torus(case["l1"], case["l2"])
        marks = sorted({int(x) for x in rng.integers(g.n, size=case["marks"])})
        return "ctqw", g, dict(gamma=0.25, dt=case["dt"], taylor_order=case["K"], marked=marks), _random(g.n, seed), case["steps"]
    if k == "regular":
        g = _regular(case["n"], case["d"], seed)
        dt, horizon = _search(g.n, case["d"])
        psi = _uniform(g.n) * np.exp(0.01j * rng.standard_normal(g.n))
        return "ctqw", g, dict(gamma=1.0 / case["d"], dt=dt, trunc_tol=1e-8, horizon_steps=horizon,
                               marked=[int(rng.integers(g.n))]), psi, case["steps"]
    if k == "hypercube":
        g = I.hypercube(case["dim"])
        return "coined", g, dict(marked=[int(rng.integers(g.n))]), _uniform(g.n_arcs), case["steps"]
    if k == "gridwalk":
        g = I.torus(case["l1"], case["l2"])
        return "coined", g, dict(marked=[int(rng.integers(g.n))]), _uniform(g.n_arcs), case["steps"]
    if k == "irregular":
        g = _sparse_graph(case["n"], case["deg"], seed)
        return "coined", g, dict(marked=[int(rng.integers(g.n))]), _random(g.n_arcs, seed), case["steps"]
    if k == "lattice":
        g = I.torus_directed(case["l1"], case["l2"])
        return "coined", g, dict(coin="fourier", shift="persistent"), _random(g.n_arcs, seed), case["steps"]
    if k == "dense":
        g = I.complete(case["n"])
        psi = np.repeat(_uniform(g.n)[:, None], case["columns"], axis=1)
        psi = psi * np.exp(0.2j * rng.standard_normal(psi.shape))
        return "ctqw", g, dict(gamma=1.0 / g.n, dt=case["dt"], taylor_order=case["K"], layout="dense", columns=case["columns"],
                               marked=[int(rng.integers(g.n))]), psi.reshape(-1), case["steps"]
    raise ValueError(f"{k} {dtype}")


def _sparse(case, seed):
    g = _sparse_graph(case["n"], case["deg"], seed)
    gamma = 1.0 / case["deg"]
    h = gamma * int(np.diff(g.row_ptr).max()) + 1.0
    mark = seed % g.n
    return g, gamma, case["dt"] / h, mark, range(case["every"], case["every"] * case["count"] + 1, case["every"])


def prepare(case, seed):
    k, dtype = case["kind"], case["dtype"]
    td = torch.complex128 if dtype == "c128" else torch.complex64
    if k == "small":
        walks = _small_walks(case, seed)
        plans = [Plan(g, kind, dtype=dtype, **kw) for kind, g, kw, _, _ in walks]
        flat, states, at = torch.zeros(sum(p.state_len + 1 for p in plans), dtype=td, device="cuda"), [], 0
        for p, w in zip(plans, walks):
            states.append(flat[at:at + p.state_len])
            states[-1].copy_(torch.from_numpy(w[3]))
            at += (p.state_len + 1) // 2 * 2
        return dict(case=case, plans=plans, flat=flat, states=states, steps=[w[4] for w in walks])
    if k == "batch":
        walks = _batch_walks(case, seed)
        plans = [Plan(g, "ctqw", dtype=dtype, layout="structured", gamma=1.0 / d, dt=dt, trunc_tol=1e-8,
                      horizon_steps=horizon, marked=[m]) for g, d, dt, horizon, m in walks]
        flat, states, at = torch.zeros(sum(p.state_len + 1 for p in plans), dtype=td, device="cuda"), [], 0
        for p in plans:
            states.append(flat[at:at + p.state_len])
            states[-1].fill_(1.0 / math.sqrt(p.state_len))
            at += (p.state_len + 1) // 2 * 2
        tiles = 16 * sum(p.state_len // 256 + 8 for p in plans)
        return dict(case=case, plans=plans, flat=flat, states=states, batch=Batch(len(plans), tiles, dtype),
                    hist=torch.zeros((len(plans), case["steps"]), dtype=torch.float64, device="cuda"))
    if k == "sparse":
        g, gamma, dt, mark, steps = _sparse(case, seed)
        w = ContinuousTime(g, gamma, dt, marked=[mark], dtype=dtype, trunc_tol=1e-13, horizon_steps=1000)
        return dict(case=case, walk=w, psi=w.plan.state(_uniform(g.n)), steps=steps)
    if k == "squares":
        g, tess = I.stag_lattice(case["l1"], case["l2"])
        mark = int(np.random.default_rng([seed, 5]).integers(g.n))
        w = Staggered(g, tess, marked=[mark], dtype=dtype)
        return dict(case=case, plan=w.plan, psi=w.plan.state(_uniform(g.n)), steps=case["steps"])
    kind, g, kw, psi, steps = _walk(case, seed)
    plan = Plan(g, kind, dtype=dtype, **kw)
    return dict(case=case, plan=plan, psi=plan.state(psi), steps=steps)


def run(state):
    k = state["case"]["kind"]
    if k == "small":
        state["desc"] = evolve_many(state["plans"], state["states"], state["steps"])
        return state["flat"]
    if k == "batch":
        b, steps = state["batch"], state["case"]["steps"]
        state["hist"].zero_()
        for i, (p, psi) in enumerate(zip(state["plans"], state["states"])):
            b.set_slot(i, p, psi, steps, hist=state["hist"][i])
        b.commit()
        b.run_to_completion()
        return state["flat"], state["hist"]
    if k == "sparse":
        return state["walk"].simulate(state["steps"], state["psi"])
    p, norm, pm = state["plan"].evolve(state["psi"], state["steps"], readout=True)
    return state["psi"], p, norm, pm


def _sizes(case):
    """(state elements, vertices, arcs, steps) summed over a case's walks."""
    k = case["kind"]
    if k == "cycle":
        return 2 * case["n"], case["n"], 2 * case["n"], case["steps"]
    if k == "small":
        n = case["count"] * (case["nmax"] - 24) / math.log(case["nmax"] / 24.0)
        return 2.4 * n, n, 4.4 * n, 0.75 * case["steps"]
    if k == "batch":
        n = case["count"] * (case["nmax"] - case["nmin"]) / math.log(case["nmax"] / case["nmin"])
        return n, n, 5.5 * n, case["steps"]
    if k in ("sparse", "irregular"):
        a = case["n"] * case["deg"]
        return (case["n"], case["n"], a, case["every"] * case["count"]) if k == "sparse" else (a, case["n"], a, case["steps"])
    if k == "regular":
        return case["n"], case["n"], case["n"] * case["d"], case["steps"]
    if k == "hypercube":
        n = 1 << case["dim"]
        return n * case["dim"], n, n * case["dim"], case["steps"]
    if k == "dense":
        return case["n"] * case["columns"], case["n"] * case["columns"], case["n"] * (case["n"] - 1), case["steps"]
    n = case["l1"] * case["l2"]
    return (n, n, 4 * n, case["steps"]) if k in ("grid", "squares") else (4 * n, n, 4 * n, case["steps"])


def work(case):
    """State in and out once, the probabilities written, the neighbour table read once
    where the graph is irregular; and one application of the step's operator per step
    (a multiply and an add on each real part of each arc's amplitude)."""
    length, n, arcs, steps = _sizes(case)
    e = 16 if case["dtype"] == "c128" else 8
    k = case["kind"]
    out = case["count"] if k == "sparse" else 1
    table = 4 * arcs if k in ("sparse", "regular", "batch", "irregular", "small") else 0
    if k == "dense":
        return {"bytes": 2 * e * length + 8 * n + e / 2 * case["n"] ** 2, "flops": 4.0 * arcs * case["columns"] * steps}
    probs = 0 if k in ("small", "batch", "sparse") else 8 * n
    return {"bytes": (1 + out) * e * length + probs + table, "flops": 4.0 * arcs * steps}


# ---- the same in 64 bits ------------------------------------------------------

def _on(x):
    return torch.as_tensor(x, device="cuda" if torch.cuda.is_available() else "cpu")


def _tails(g):
    return np.repeat(np.arange(g.n, dtype=np.int64), np.diff(g.row_ptr))


def _reverse(g):
    t, h = _tails(g), g.col.astype(np.int64)
    rev = np.empty(t.size, dtype=np.int64)
    rev[np.lexsort((t, h))] = np.lexsort((h, t))
    return rev


def _sum_at(x, index, n):
    out = torch.zeros((n, 2), dtype=torch.float64, device=x.device)
    out.index_add_(0, index, torch.view_as_real(x))
    return torch.view_as_complex(out)


def _exact_ctqw(g, psi, gamma, dt, K, marked, stops):
    """The order-K Taylor propagator in power form, the states after each of `stops`."""
    d = np.diff(g.row_ptr)
    psi, out = _on(psi.astype(np.complex128)), []
    mk = _on(np.asarray(marked, dtype=np.int64))
    regular = d.min() == d.max()
    col = _on(g.col.astype(np.int64))
    cols = col.view(g.n, -1).t().contiguous() if regular else None
    tails = None if regular else _on(_tails(g))
    for s in range(1, max(stops) + 1):
        term, acc = psi, psi.clone()
        for k in range(1, K + 1):
            nb = sum(term[c] for c in cols) if regular else _sum_at(term[col], tails, g.n)
            h = -gamma * nb
            h[mk] -= term[mk]
            term = h * (-1j * dt / k)
            acc += term
        psi = acc
        if s in stops:
            out.append(psi)
    return out


def _exact_coined(g, psi, kw, steps):
    psi = _on(psi)
    mk = torch.zeros(g.n, dtype=torch.bool)
    mk[torch.as_tensor(kw.get("marked", []), dtype=torch.int64)] = True
    mk = mk.to(psi.device)
    coin = kw.get("coin", "grover")
    tails_np = _tails(g)
    tails, rev, deg = _on(tails_np), _on(_reverse(g)), _on(np.diff(g.row_ptr).astype(np.float64))
    amk = mk[tails]
    if coin in ("hadamard", "fourier"):
        d = int(g.row_ptr[1])
        j = np.arange(d)
        f = np.exp(2j * np.pi * ((j[:, None] * j[None, :]) % d) / d) / math.sqrt(d)
        f = _on(f)
    if kw.get("shift") == "persistent":
        # slot j of v comes from slot j of the vertex one step against direction j
        heads = g.col.reshape(g.n, -1).astype(np.int64)
        src = np.empty_like(heads)
        for j in range(heads.shape[1]):
            src[heads[:, j], j] = np.arange(g.n, dtype=np.int64) * heads.shape[1] + j
        move = _on(src.reshape(-1))
    else:
        move = rev
    for _ in range(steps):
        if coin in ("hadamard", "fourier"):
            x = psi.view(g.n, -1)
            y = torch.stack([sum(f[a, b] * x[:, b] for b in range(x.shape[1])) for a in range(x.shape[1])], 1).reshape(-1)
        else:
            m = _sum_at(psi, tails, g.n) / deg.clamp(min=1.0)
            y = 2.0 * m[tails] - psi
        y = torch.where(amk, -psi, y)
        psi = y[move]
    return psi


def _exact_staggered(g, tess, psi, marked, steps):
    psi = _on(psi)
    polys = [_on(t.poly_vert.reshape(t.n_polygons, -1).astype(np.int64)) for t in tess]
    mk = _on(np.asarray(marked, dtype=np.int64))
    for _ in range(steps):
        psi = psi.clone()
        psi[mk] = -psi[mk]
        for p in polys:
            x = psi[p]
            new = torch.empty_like(psi)
            new[p] = 2.0 * x.mean(dim=1, keepdim=True) - x
            psi = new
    return psi


def _readout(psi, arcs_of, marked):
    q = psi.real ** 2 + psi.imag ** 2
    if arcs_of is not None:
        tails, n = arcs_of
        q = torch.zeros(n, dtype=torch.float64, device=q.device).index_add_(0, tails, q)
    return psi, q, q.sum(), q[_on(np.asarray(marked, dtype=np.int64))].sum()


def _flat(parts):
    """The walks' states as prepare() lays them out, each at an even element."""
    out, at = torch.zeros(sum(x.numel() + 1 for x in parts), dtype=torch.complex128), 0
    for x in parts:
        out[at:at + x.numel()] = x.cpu()
        at += (x.numel() + 1) // 2 * 2
    return out


def _one(kind, g, kw, psi, steps):
    if kind == "coined":
        return _exact_coined(g, psi, kw, steps)
    if kind == "staggered":
        return _exact_staggered(g, kw["tessellations"], psi, kw["marked"], steps)
    return _exact_ctqw(g, psi, kw["gamma"], kw["dt"], kw.get("taylor_order", 30), kw.get("marked", []), [steps])[0]


def exact(case, seed):
    k = case["kind"]
    if k == "small":
        return _flat([_one(*w) for w in _small_walks(case, seed)])
    if k == "batch":
        states, hist = [], []
        for g, d, dt, _, m in _batch_walks(case, seed):
            got = _exact_ctqw(g, _uniform(g.n), 1.0 / d, dt, 24, [m], list(range(1, case["steps"] + 1)))
            states.append(got[-1])
            hist.append(torch.stack([x[m].abs() ** 2 for x in got]).cpu())
        return _flat(states), torch.stack(hist)
    if k == "sparse":
        g, gamma, dt, mark, steps = _sparse(case, seed)
        return _exact_ctqw(g, _uniform(g.n), gamma, dt, 24, [mark], list(steps))
    if k == "squares":
        g, tess = I.stag_lattice(case["l1"], case["l2"])
        mark = int(np.random.default_rng([seed, 5]).integers(g.n))
        return _readout(_exact_staggered(g, tess, _uniform(g.n), [mark], case["steps"]), None, [mark])
    kind, g, kw, psi, steps = _walk(case, seed)
    if k == "dense":
        # H = -gamma (J - I) - |m><m|: a stage is a column sum and a diagonal
        x = _on(psi.reshape(g.n, case["columns"]))
        for _ in range(steps):
            term, acc = x, x.clone()
            for j in range(1, kw["taylor_order"] + 1):
                h = -kw["gamma"] * (term.sum(dim=0, keepdim=True) - term)
                h[kw["marked"]] -= term[kw["marked"]]
                term = h * (-1j * kw["dt"] / j)
                acc += term
            x = acc
        q = (x.real ** 2 + x.imag ** 2)
        return x.reshape(-1), q.reshape(-1), q.sum(), q[kw["marked"]].sum()
    if kind == "coined":
        return _readout(_exact_coined(g, psi, kw, steps), (_on(_tails(g)), g.n), kw.get("marked", []))
    return _readout(_one(kind, g, kw, psi, steps), None, kw.get("marked", []))
