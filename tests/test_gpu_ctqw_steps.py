"""A CTQW's time steps are the same wherever a call or a launch ends: evolve(a)
then evolve(b) has the bits of evolve(a + b), a batched walk those of the same
walk alone, on every path and in both types; and amplitudes far out in the tail
of a spreading walk keep their own relative accuracy, not the state's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_08186_amd import inputs as I

pytestmark = pytest.mark.gpu

WALKS = {  # graph, layout, columns, expected structure
    "small": (I.erdos_renyi(300, 0.02, seed=2), "auto", 0, "small"),
    "general": (I.erdos_renyi(2500, 7 / 2499, seed=3), "csr", 0, "general"),
    "ell": (I.random_regular(3000, 5, seed=4), "structured", 0, "ell"),
    "cycle": (I.cycle(501), "structured", 0, "cycle"),
    "hypercube": (I.hypercube(9), "structured", 0, "hypercube"),
    "torus": (I.torus(30, 41), "structured", 0, "torus"),
    "sweep": (I.torus(96, 130), "structured", 0, "torus"),
    "dense": (I.erdos_renyi(300, 0.2, seed=5), "dense", 1, "dense"),
    "dense_40": (I.erdos_renyi(300, 0.2, seed=5), "dense", 40, "dense"),
}


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("name", list(WALKS))
def test_split_calls_equal_one_call(name, dtype):
    from paper_2406_08186_amd.walk import Plan
    g, layout, columns, structure = WALKS[name]
    print(f"[case] split calls {name} {dtype}", flush=True)
    pl = Plan(g, "ctqw", dtype=dtype, layout=layout, gamma=1.0 / int(np.diff(g.row_ptr).max()), dt=0.1,
              taylor_order=12, marked=[1, g.n - 2], columns=columns)
    assert pl.structure == structure
    psi0 = I.random_state(pl.state_len, 8)
    whole = pl.state(psi0)
    pl.evolve(whole, 71)
    for cuts in ((16, 55), (20, 43, 8), (70, 1)):
        parts = pl.state(psi0)
        for m in cuts:
            pl.evolve(parts, m)
        torch.cuda.synchronize()
        assert torch.equal(whole, parts), cuts


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_batched_walk_equals_the_walk_alone(dtype):
    from paper_2406_08186_amd.walk import Batch, Plan
    g = I.random_regular(9000, 6, seed=11)
    print(f"[case] batch of one and evolve, {dtype}", flush=True)
    pl = Plan(g, "ctqw", dtype=dtype, layout="structured", gamma=1 / 6, dt=0.5, taylor_order=11, marked=[7])
    alone, batched = (pl.state(I.random_state(g.n, 1)) for _ in range(2))
    pl.evolve(alone, 37)
    b = Batch(1, 64, dtype)
    b.set_slot(0, pl, batched, 37)
    b.commit()
    b.run_to_completion()
    torch.cuda.synchronize()
    assert torch.equal(alone, batched)


@pytest.mark.parametrize("shape,steps,gamma,dt,K", [((201,), 16, 0.5, 1.0, 13), ((2001,), 16, 0.5, 1.0, 13),
                                                   ((96, 80), 16, 0.25, 0.5, 12), ((96, 140), 64, 0.25, 0.1, 20),
                                                   ((8, 400), 32, 0.25, 0.86, 13)])
def test_tail_amplitudes(shape, steps, gamma, dt, K):
    """One vertex excited.  At distances beyond twice the front's along every axis of more than 8
    vertices an amplitude is a sum of terms that fall quickly and do not cancel, so `steps` Horner
    schemes of K stages of a few roundings each leave it 4 K steps 2^-53 < 1e-12 of itself."""
    from paper_2406_08186_amd.walk import Plan
    print(f"[case] tail {shape} steps {steps}", flush=True)
    g = I.cycle(shape[0]) if len(shape) == 1 else I.torus(*shape)
    pl = Plan(g, "ctqw", dtype="c128", layout="structured", gamma=gamma, dt=dt, taylor_order=K)
    psi0 = np.zeros(g.n, np.complex128)
    psi0[0] = 1.0
    psi = pl.state(psi0)
    p, _, _ = pl.evolve(psi, steps, readout=True)
    torch.cuda.synchronize()
    got, p = psi.cpu().numpy(), p.cpu().numpy()
    ref = oracle.ctqw_evolve(g.row_ptr, g.col, psi0, steps, gamma=gamma, dt=dt, K=K)
    assert np.abs(got - ref).max() < 1e-12
    tail = np.ones(shape, bool)
    for axis, l in enumerate(shape):
        if l > 8:
            d = np.minimum(np.arange(l), l - np.arange(l))
            far = (d > 2 * (2 * gamma * dt * steps)) & (d < l // 2 - 2)
            tail &= far.reshape([-1 if a == axis else 1 for a in range(len(shape))])
        else:
            tail &= (np.arange(l) == 0).reshape([-1 if a == axis else 1 for a in range(len(shape))])
    tail = tail.reshape(-1)
    assert tail.any() and np.abs(ref[tail]).min() < 1e-13
    assert (np.abs(got - ref)[tail] <= 1e-12 * np.abs(ref)[tail]).all()
    tail &= np.abs(ref) > 1e-150  # their squares are normal numbers
    assert (np.abs(p - np.abs(ref) ** 2)[tail] <= 1e-11 * np.abs(ref)[tail] ** 2).all()
