"""Coined walks in CSR order, whose steps leave the shift to the next step's
reads: the same bits as single steps for odd and even counts, with vertices
above a tile's arcs, of degree zero and one, marked and not; and the oracle's
state."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_08186_amd import inputs as I

pytestmark = pytest.mark.gpu


def _graph(n, hub, seed):
    """A random graph of mean degree about 6 on the first n - 3 vertices, vertex 5
    joined to `hub` others."""
    r = np.random.default_rng(seed)
    e = {(min(a, b), max(a, b)) for a, b in r.integers(0, n - 3, (3 * n, 2)) if a != b}
    e |= {(min(5, b), max(5, b)) for b in r.choice(n - 3, hub, replace=False) if b != 5}
    e = np.array(sorted(e))
    src, dst = np.concatenate([e[:, 0], e[:, 1]]), np.concatenate([e[:, 1], e[:, 0]])
    o = np.lexsort((dst, src))
    rp = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))])
    return rp.astype(np.int64), dst[o].astype(np.int32)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,hub,marked", [(40, 3, [0, 39]), (700, 20, []), (3000, 2048, [5, 17]), (3000, 2900, [])])
def test_steps_equal_single_steps(n, hub, marked, dtype):
    from paper_2406_08186_amd.walk import Plan
    print(f"[case] coined CSR n {n} hub {hub} {dtype}", flush=True)
    rp, col = _graph(n, hub, n + hub)
    g = I.Graph(n, rp, col)
    pl = Plan(g, "coined", dtype=dtype, layout="csr", marked=marked)
    assert pl.structure == "general"
    psi0 = I.random_state(len(col), 2)
    single = pl.state(psi0)
    for steps in range(1, 6):
        pl.evolve(single, 1)
        got = pl.state(psi0)
        pl.evolve(got, steps)
        torch.cuda.synchronize()
        assert torch.equal(got, single), steps
    ref = oracle.coined_evolve(rp, col, psi0, 5, marked=marked)
    err = got.cpu().numpy().astype(np.complex128) - ref
    assert (np.abs(err).max() < 1e-12) if dtype == "c128" else (np.linalg.norm(err) < 1e-5)
