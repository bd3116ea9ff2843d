"""Whole groups of CTQW time steps evaluated as one Chebyshev series
(complex128): the same polynomial T_K(-i dt H)^m, so every result equals the
oracle's step-by-step one to 1e-12, at step counts around the group size, at
short Taylor orders (where T_K is far from exp), at step lengths whose groups
are shorter, and on every path that takes groups.  complex64 walks take single
steps, whatever the count."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_08186_amd import inputs as I

pytestmark = pytest.mark.gpu


def _check(g, steps, layout, gamma, dt, K, marked, columns=0, structure=None):
    from paper_2406_08186_amd.walk import Plan
    print(f"[case] series {g.name} {layout} K={K} dt={dt} steps={steps}", flush=True)
    pl = Plan(g, "ctqw", dtype="c128", layout=layout, gamma=gamma, dt=dt, taylor_order=K, marked=marked,
              columns=columns)
    assert structure is None or pl.structure == structure
    nb = max(1, columns)
    psi0 = np.stack([I.random_state(g.n, steps + K + b) for b in range(nb)], axis=1)
    psi = pl.state(psi0.reshape(-1))
    p, norm, pm = pl.evolve(psi, steps, readout=True)
    torch.cuda.synchronize()
    got = psi.cpu().numpy().astype(np.complex128).reshape(g.n, nb)
    p = p.cpu().numpy().reshape(g.n, nb)
    for b in range(nb):
        ref = oracle.ctqw_evolve(g.row_ptr, g.col, psi0[:, b], steps, gamma=gamma, dt=dt, K=K, marked=marked)
        pref = np.abs(ref) ** 2
        assert np.abs(got[:, b] - ref).max() < 1e-12
        assert np.abs(p[:, b] - pref).max() < 1e-12
    assert abs(float(norm) - p.sum()) < 1e-9 and abs(float(pm) - p[marked].sum()) < 1e-9


GRAPHS = {
    "general": (I.erdos_renyi(2500, 7 / 2499, seed=3), "csr"),       # with isolated vertices
    "general_long": (I.random_mixed(300, seed=5), "csr"),             # a hub, many lanes per row
    "ell": (I.random_regular(3000, 5, seed=4), "structured"),
    "cycle": (I.cycle(501), "structured"),
    "hypercube": (I.hypercube(9), "structured"),
    "torus": (I.torus(30, 41), "structured"),                        # too narrow for the blocked sweep
}


@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("steps,rho,K", [(8, 0.3, 12), (15, 1.0, 13), (16, 1.0, 13), (33, 0.1, 20), (31, 0.7, 3),
                                         (17, 3.0, 24), (9, 20.0, 64)])
def test_series_matches_oracle(name, steps, rho, K):
    g, layout = GRAPHS[name]
    gamma = 1.0 / int(np.diff(g.row_ptr).max())
    # rho = dt (gamma d_max + 1 for the marks); 20 is beyond any series and stays on single stages
    _check(g, steps, layout, gamma, rho / 2.0 if rho <= 10 else 2.0, K, [1, g.n - 2],
           structure=name.split("_")[0])


def test_series_sliced_paths():
    """Vectors above 7.5 MiB: the column-sliced ELL and CSR stages inside a group."""
    for g, layout in ((I.random_regular(990000, 3, seed=6), "structured"), (I.erdos_renyi(1000001, 5e-6, seed=7), "csr")):
        _check(g, 17, layout, 0.1, 0.3, 7, [5, g.n - 1])


@pytest.mark.parametrize("columns", [1, 5, 40])
@pytest.mark.parametrize("n,steps,rho,K", [(130, 16, 1.0, 13), (700, 26, 0.4, 4)])
def test_series_dense(columns, n, steps, rho, K):
    g = I.erdos_renyi(n, 0.3, seed=9)
    _check(g, steps, "dense", 1.0 / int(np.diff(g.row_ptr).max()), rho / 2.0, K, [3, n - 1], columns, "dense")


@pytest.mark.parametrize("l1,l2", [(96, 80), (17, 64), (64, 65), (50, 130), (300, 64)])
@pytest.mark.parametrize("steps,rho,K", [(8, 0.1, 20), (71, 0.2, 7), (64, 0.1, 20), (40, 1.0, 13), (19, 2.0, 6)])
def test_series_grid_sweep(l1, l2, steps, rho, K):
    """Blocked series: strips clamped at ragged edges, windows that wrap, marks on strip edges,
    one and several launches, Taylor orders that the blocked single steps divide and do not."""
    g = I.torus(l1, l2)
    marked = sorted({0, 8 * l2 + 53, 13 * l2 + 54, g.n - 1})
    _check(g, steps, "structured", 0.25, rho / 2.0, K, marked, structure="torus")
    if l1 == 96:
        _check(g, steps, "structured", 0.25, rho, K, [], structure="torus")


def test_series_groups_are_resumable():
    """evolve(16 a) then evolve(b) equals evolve(16 a + b) bitwise; complex64: any split."""
    from paper_2406_08186_amd.walk import Plan
    for name in ("general", "ell"):
        g, layout = GRAPHS[name]
        for dtype in ("c128", "c64"):
            pl = Plan(g, "ctqw", dtype=dtype, layout=layout, gamma=0.1, dt=0.5, taylor_order=11, marked=[4])
            a, b = (pl.state(I.random_state(g.n, 8)) for _ in range(2))
            pl.evolve(a, 43)
            for part in (32, 11) if dtype == "c128" else (20, 23):
                pl.evolve(b, part)
            torch.cuda.synchronize()
            assert torch.equal(a, b)


def _ring_plus(n, d, seed):
    """A cycle with a d-2-regular random graph over it (degree <= d), d >= 2."""
    v = np.arange(n)
    e = [np.stack([v, (v + 1) % n], 1)]
    if d > 2:
        rng = np.random.default_rng(seed)
        for _ in range(d - 2):
            p = rng.permutation(n)[: n // 2 * 2].reshape(-1, 2)
            e.append(p)
    e = np.sort(np.concatenate(e), axis=1)
    return I.from_edges(n, np.unique(e, axis=0), f"ring{n}d{d}")


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,d,steps,rho,K", [(4, 2, 16, 0.5, 9), (63, 4, 37, 1.0, 13), (1023, 3, 16, 0.2, 6),
                                             (1025, 6, 33, 1.0, 12), (1030, 15, 18, 0.7, 11), (1600, 9, 17, 0.4, 10),
                                             (2049, 5, 16, 1.0, 13), (2500, 3, 20, 0.3, 2), (90, 16, 40, 2.0, 20), (200, 32, 17, 1.0, 13),
                                             (200, 33, 17, 1.0, 13), (1400, 24, 16, 1.0, 13)])
def test_small_walk_registers(n, d, steps, rho, K, dtype):
    """The one-workgroup walk with its tables in registers: one, two and four vertices per
    thread, rows padded to 4, 8 and up to 32, degrees beyond, whole groups and single steps, alone and in one
    launch with others."""
    from paper_2406_08186_amd.walk import Plan, evolve_many
    g = _ring_plus(n, d, n)
    marked = [0, n - 1]
    gamma = 1.0 / int(np.diff(g.row_ptr).max())
    print(f"[case] small registers {g.name} {dtype} steps={steps} K={K}", flush=True)
    pl = Plan(g, "ctqw", dtype=dtype, gamma=gamma, dt=rho / 2.0, taylor_order=K, marked=marked)
    es = 16 if dtype == "c128" else 8
    fits = 3 * es * n + 4 * (n + 1 + g.n_arcs) + 4 * ((n + 31) // 32) <= 156 * 1024
    assert pl.structure == ("small" if fits else "cycle" if d == 2 else "general")
    psi0 = I.random_state(n, steps)
    psi = pl.state(psi0)
    p, norm, pm = pl.evolve(psi, steps, readout=True)
    torch.cuda.synchronize()
    ref = oracle.ctqw_evolve(g.row_ptr, g.col, psi0, steps, gamma=gamma, dt=rho / 2.0, K=K, marked=marked)
    got = psi.cpu().numpy().astype(np.complex128)
    if dtype == "c128":
        assert np.abs(got - ref).max() < 1e-12
        assert np.abs(p.cpu().numpy() - np.abs(ref) ** 2).max() < 1e-12
    else:
        assert np.linalg.norm(got - ref) < 1e-5
    if pl.structure == "small":
        other = Plan(I.torus(30, 31), "ctqw", dtype=dtype, gamma=0.25, dt=0.1, taylor_order=8)
        many = [pl.state(psi0), other.state(I.random_state(930, 1))]
        desc = evolve_many([pl, other], many, [steps, 5])
        torch.cuda.synchronize()
        assert torch.equal(many[0], psi)
        del desc
