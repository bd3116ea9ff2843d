"""Dense H: walks that share H with many others are as accurate as with few."""
import numpy as np
import pytest
import torch

from paper_2406_08186_amd import inputs as I

pytestmark = pytest.mark.gpu


def _exact(psi, mark, gamma, dt, K, steps):
    """The complete graph's walk in 80 bits: a stage is a column sum and a diagonal."""
    x = psi.astype(np.clongdouble)
    c = np.longdouble(gamma)
    for _ in range(steps):
        term, acc = x, x.copy()
        for k in range(1, K + 1):
            h = -c * (term.sum(axis=0, keepdims=True) - term)
            h[mark] -= term[mark]
            term = h * (-1j * np.longdouble(dt) / k)
            acc = acc + term
        x = acc
    return x


def test_wide_blocks_err_no_more_than_narrow_ones():
    """The same 16 walks alone (the LDS-staged kernel, short k ranges) and in a block of 20 (the
    register-fed one, whose ranges are longer): root mean square errors over 64 walks.  They differ
    in the order of sums alone, and with 64 walks of 2500 entries by 1% from sampling."""
    from paper_2406_08186_amd.walk import Plan
    n, mark, kw = 2500, 7, dict(gamma=1 / 2500, dt=0.65, taylor_order=24)
    g, sums = I.complete(n), {}
    plans = {b: Plan(g, "ctqw", dtype="c128", layout="dense", columns=b, marked=[mark], **kw) for b in (16, 20)}
    for seed in range(4):
        print(f"[case] dense error, seed {seed}", flush=True)
        rng = np.random.default_rng(seed)
        psi0 = np.exp(0.2j * rng.standard_normal((n, 20))) / np.sqrt(n)
        ref = _exact(psi0[:, :16], mark, kw["gamma"], kw["dt"], 24, 8)
        for b, pl in plans.items():
            psi = pl.state(np.ascontiguousarray(psi0[:, :b]).reshape(-1))
            pl.evolve(psi, 8)
            torch.cuda.synchronize()
            err = psi.cpu().numpy().reshape(n, b)[:, :16] - ref
            sums[b] = sums.get(b, 0.0) + float((np.abs(err) ** 2).sum())
    print("rms error per walk", {b: (s / 64) ** 0.5 for b, s in sums.items()}, flush=True)
    assert sums[20] ** 0.5 < 1.02 * sums[16] ** 0.5
