"""CTQW on the CSR path with many lanes per row: the oracle's states on either
side of the vertex counts where a lane's arcs stop being in flight together."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_08186_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,degree", [(16384, 60), (16385, 60), (8192, 120), (8193, 120), (4096, 230), (4097, 230),
                                      (300, 60)])
def test_lanes_per_row(n, degree, dtype):
    from paper_2406_08186_amd.walk import Plan
    print(f"[case] CSR {n} vertices of mean degree {degree} {dtype}", flush=True)
    g = I.erdos_renyi(n, degree / (n - 1), seed=n)
    gamma = 1.0 / int(np.diff(g.row_ptr).max())
    pl = Plan(g, "ctqw", dtype=dtype, layout="csr", gamma=gamma, dt=0.6, taylor_order=9, marked=[3, n - 1])
    assert pl.structure == "general"
    psi0 = I.random_state(n, degree)
    psi = pl.state(psi0)
    p, norm, pm = pl.evolve(psi, 2, readout=True)
    torch.cuda.synchronize()
    ref = oracle.ctqw_evolve(g.row_ptr, g.col, psi0, 2, gamma=gamma, dt=0.6, K=9, marked=[3, n - 1])
    err = psi.cpu().numpy().astype(np.complex128) - ref
    assert (np.abs(err).max() < 1e-12) if dtype == "c128" else (np.linalg.norm(err) < 1e-5)
    assert np.abs(p.cpu().numpy() - np.abs(ref) ** 2).max() < (1e-12 if dtype == "c128" else 1e-6)
