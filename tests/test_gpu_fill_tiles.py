"""The block fill at the edges of its triangle tiles and of its near region:
meshes of one, two and several tiles per state, rectangular extents, extents
inside the extraction radius, and both halves of the displacement set."""
import numpy as np
import pytest

from gpu_common import FREQ, K
from oracle import efie
from workloads.mesh import connected_unit, macro_unit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the bound of the fill's other comparisons with the oracle: the closed-form
# potentials of a neighbouring cell lose four digits in both (the one-thread-
# per-entry fill and this one are 1.4e-12 off the oracle there, alike)
TOL = 1e-11


# ncell 1: 2 triangles, 1 RWG a state; 3: 18 triangles; 4: 32, one full tile;
# 5: 50 triangles, 65 RWG, tiles cut inside a state
@pytest.mark.parametrize("ncell,Dx,Dy,radius,dtype", [
    (1, 0, 0, 1, "c128"), (3, 2, 1, 1, "c128"), (3, 3, 0, 0, "c128"), (4, 0, 3, 1, "c64"), (4, 1, 1, 2, "c128"),
    (5, 2, 2, 1, "c128"), (5, 3, 1, 0, "c64")])
def test_fill_against_oracle(ncell, Dx, Dy, radius, dtype):
    from paper_2112_05082_amd import r3m
    unit = macro_unit((0.006, 0.009), ncell)
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit, FREQ, radius)
    c64 = dtype == "c64"
    out = torch.full(((2 * Dx + 1) * (2 * Dy + 1), geom.n, geom.n), float("nan"),
                     dtype=torch.complex64 if c64 else torch.complex128, device="cuda:0")
    r3m.r3m_fill_unique_blocks(ctx, geom, Dx, Dy, r3m.C64 if c64 else r3m.C128, out)
    got = out.cpu().numpy()
    # complex64 storage rounds to 6e-8
    tol = 2e-7 if c64 else TOL
    for dy in range(-Dy, Dy + 1):
        for dx in range(-Dx, Dx + 1):
            ref = efie.displacement_block(unit, dx, dy, K, radius)
            blk = got[(dy + Dy) * (2 * Dx + 1) + dx + Dx]
            assert np.abs(blk - ref).max() <= tol * np.abs(ref).max(), (dx, dy)
    ctx.close()


def test_fill_connected_far_and_near():
    """Shared bases that bridge two cells: the near region grows by their reach."""
    from paper_2112_05082_amd import r3m
    cu = connected_unit((0.006, 0.009))
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_connected(cu, FREQ, 1)
    D = 4
    out = torch.full(((2 * D + 1) ** 2, geom.n, geom.n), float("nan"), dtype=torch.complex128, device="cuda:0")
    r3m.r3m_fill_unique_blocks(ctx, geom, D, D, r3m.C128, out)
    got = out.cpu().numpy()
    for dx, dy in ((4, -1), (-4, 1), (3, 0), (-3, -2), (2, 2), (0, -4)):
        def mesh(c):
            px, py = cu.period
            return efie.rwg_mesh(cu.vert, cu.tri, cu.rwg, (c[0] * px, c[1] * py, 0.0), c, cu.tri_cell, cu.state_off)
        ref = efie.efie_matrix(mesh((dx, dy)), mesh((0, 0)), K, 1)
        blk = got[(dy + D) * (2 * D + 1) + dx + D]
        assert np.abs(blk - ref).max() <= TOL * np.abs(ref).max(), (dx, dy)
    ctx.close()
