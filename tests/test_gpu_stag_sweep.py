"""Staggered walks on the square lattice, several steps per launch: the same
bits whatever the steps of a launch, in both forms, at lattices smaller than a
wavefront's window, ragged strips in both directions, marks on strip edges; and
equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_08186_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("form", ["reflection", "hamiltonian"])
@pytest.mark.parametrize("l1,l2", [(4, 4), (4, 130), (30, 104), (26, 112), (258, 106), (70, 250)])
def test_sweep_equals_single_steps(l1, l2, form, dtype):
    from paper_2406_08186_amd.walk import Plan
    print(f"[case] square lattice {l1}x{l2} {form} {dtype}", flush=True)
    g, tess = I.stag_lattice(l1, l2)
    if form == "hamiltonian":
        tess = [I.Tessellation(t.poly_ptr, t.poly_vert, None, a) for t, a in zip(tess, (0.83, -0.41))]
    marked = sorted({0, l2 - 1, min(103, l2 - 1) + l2, g.n // 2, g.n - 1}) if (l1 // 2) % 2 else []
    pl = Plan(g, "staggered", dtype=dtype, layout="structured", marked=marked, tessellations=tess)
    assert pl.structure == "stag_lattice"
    psi0 = I.random_state(g.n, l1 + l2)
    buf = torch.zeros(g.n + 1, dtype=pl.state(psi0).dtype, device="cuda")
    single = pl.state(psi0)
    for steps in range(1, 15):
        pl.evolve(single, 1)
        got = buf[1:] if dtype == "c64" else pl.state(psi0)  # complex64: 8-byte aligned only
        got.copy_(pl.state(psi0))
        pl.evolve(got, steps)
        torch.cuda.synchronize()
        assert torch.equal(got, single), steps
    p, norm, pm = pl.evolve(got, 7, readout=True)
    torch.cuda.synchronize()
    ref = oracle.staggered_evolve(g.n, tess, psi0, 21, marked=marked)
    err = got.cpu().numpy().astype(np.complex128) - ref
    assert (np.abs(err).max() < 1e-12) if dtype == "c128" else (np.linalg.norm(err) < 1e-5)
    assert np.abs(p.cpu().numpy() - np.abs(ref) ** 2).max() < (1e-12 if dtype == "c128" else 1e-6)
    assert abs(float(pm) - float((np.abs(ref) ** 2)[marked].sum())) < (1e-12 if dtype == "c128" else 1e-6)


def _edges(n):
    ptr, v = np.arange(0, n + 1, 2), np.arange(n)
    return I.cycle(n), [I.Tessellation(ptr, v, None, None), I.Tessellation(ptr, np.roll(v, -1), None, None)]


@pytest.mark.parametrize("name,dtype", [("64x66", "c64"), ("138x144", "c64"), ("64x66", "c128"), ("96x104", "c128"),
                                        (2050, "c64"), (19968, "c64"), (2050, "c128"), (9984, "c128")])
@pytest.mark.parametrize("form", ["reflection", "hamiltonian"])
def test_one_workgroup_more_polygons_than_threads(name, dtype, form):
    """Several polygons of two or four vertices per thread, up to the largest
    graphs the LDS holds, one and two tessellations."""
    from paper_2406_08186_amd.walk import Plan
    print(f"[case] one-workgroup staggered {name} {form} {dtype}", flush=True)
    g, tess = I.stag_lattice(*map(int, name.split("x"))) if isinstance(name, str) else _edges(name)
    if form == "hamiltonian":
        tess = [I.Tessellation(t.poly_ptr, t.poly_vert, None, a) for t, a in zip(tess, (0.83, -0.41))]
    marked = [0, 1025, g.n - 1]
    pl = Plan(g, "staggered", dtype=dtype, marked=marked, tessellations=tess)
    assert pl.structure == "small"
    psi0 = I.random_state(g.n, 3)
    x = pl.state(psi0)
    p, norm, pm = pl.evolve(x, 9, readout=True)
    torch.cuda.synchronize()
    ref = oracle.staggered_evolve(g.n, tess, psi0, 9, marked=marked)
    err = x.cpu().numpy().astype(np.complex128) - ref
    assert (np.abs(err).max() < 1e-12) if dtype == "c128" else (np.linalg.norm(err) < 1e-5)
    assert abs(float(pm) - float((np.abs(ref) ** 2)[marked].sum())) < (1e-12 if dtype == "c128" else 1e-6)
