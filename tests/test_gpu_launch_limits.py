"""Calls whose work passes what one launch takes: a grid dimension holds fewer
than 2^32 threads, and a larger launch wraps around without an error, so its
last workgroups never run."""
import numpy as np
import pytest

from gpu_common import FREQ, K
from oracle import efie
from workloads.mesh import macro_unit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_fill_of_more_blocks_than_one_launch_takes():
    """One basis, 2,897 x 2,897 displacements: 4,196,304 workgroups of 1,024
    threads for half of them (the other half are their transposes)."""
    from paper_2112_05082_amd import r3m
    unit = macro_unit((0.006,), 1)
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit, FREQ, 1)
    blocks = {}
    for D in (1448, 9):
        blocks[D] = torch.full((2 * D + 1, 2 * D + 1), float("nan"), dtype=torch.complex64, device="cuda:0")
        r3m.r3m_fill_unique_blocks(ctx, geom, D, D, r3m.C64, blocks[D])
    D, out = 1448, blocks[1448]
    assert bool(torch.isfinite(torch.view_as_real(out)).all())
    # a block does not depend on the extents
    assert torch.equal(out[D - 9:D + 10, D - 9:D + 10], blocks[9])
    # complex64 storage rounds to 6e-8; the phase of up to 6,400 rad, rounded
    # to 2^-53 of itself, to less
    for dx, dy in ((-1448, -1448), (1448, 1448), (1447, -1448), (-3, -1448), (-1448, 0), (1448, 0), (4, 1), (-700, -5)):
        ref = efie.displacement_block(unit, dx, dy, K, 1)[0, 0]
        assert abs(complex(out[dy + D, dx + D]) - ref) <= 2e-7 * abs(ref), (dx, dy)
    ctx.close()
