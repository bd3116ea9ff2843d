"""Workspace of grid CTQW plans (host only): three state buffers where stages are
blocked, two where they are not, and the readout's scratch; so the grids that the
allocation-free entry point's 64 MiB hold follow from their size alone."""
import pytest

from paper_2406_08186_amd import inputs as I
from paper_2406_08186_amd.walk import Plan


def _up(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("dtype,size", [("c64", 8), ("c128", 16)])
@pytest.mark.parametrize("l1,l2,K", [(30, 41, 12), (96, 130, 20), (8, 400, 13), (1024, 1024, 20), (1080, 1097, 20),
                                     (1024, 1030, 13)])
def test_grid_workspace(l1, l2, K, dtype, size):
    pl = Plan(I.torus(l1, l2), "ctqw", dtype=dtype, layout="structured", gamma=0.25, dt=0.2, taylor_order=K,
              upload=False)
    n = l1 * l2
    need = (3 if pl.info.block_depth > 1 else 2) * _up(size * n) + _up(8 * n)
    assert need <= pl.info.work_bytes <= need + _up(8 * (n + 255) // 256) + 256
    if dtype == "c128" and (l1, l2) == (1080, 1097):
        assert pl.info.work_bytes <= 64 << 20  # within a MiB of it: qw_evolve_static takes this grid
