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


def test_rcs_of_more_workgroups_than_one_launch_takes():
    """8,192 right-hand sides x 65,537 directions: 16,785,408 workgroups of 256 threads."""
    from paper_2112_05082_amd import r3m
    unit = macro_unit((0.006,), 1)
    dev, B, n_dir = "cuda:0", 8192, 65537
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit, FREQ, 1)
    states = torch.zeros(1, dtype=torch.uint8, device=dev)
    batch = r3m.Batch([(1, 1)] * B, list(range(B)), [0] * B, states)
    I = torch.randn(B, dtype=torch.complex128, device=dev, generator=torch.Generator(dev).manual_seed(1))
    t = np.linspace(-1.0, 1.0, n_dir)
    dirs = np.stack([1.4 * t, 3.0 * t], 1)
    sigma = torch.full((B, n_dir), float("nan"), dtype=torch.float64, device=dev)
    r3m.r3m_rcs(ctx, geom, batch, I, dirs, 1.0, sigma)
    # one basis: sigma is |I|^2 times the pattern of a unit current
    one = torch.zeros(n_dir, dtype=torch.float64, device=dev)
    r3m.r3m_rcs(ctx, geom, r3m.Batch([(1, 1)], [0], [0], states), torch.ones(1, dtype=torch.complex128, device=dev),
                dirs, 1.0, one)
    assert bool((one > 0).all())
    for b in range(0, B, 512):
        ref = I[b:b + 512].abs().square()[:, None] * one[None, :]
        assert bool(((sigma[b:b + 512] - ref).abs() <= 1e-12 * ref).all()), b
    ctx.close()


def test_line_transforms_of_more_workgroups_than_one_launch_takes():
    """83 bases (odd: one line to a workgroup) x 128 rows x 1,600 right-hand
    sides: 16,998,400 workgroups of 256 threads a row pass."""
    from paper_2112_05082_amd import r3m
    dev, n, D, B, L = "cuda:0", 83, 63, 1600, 2
    ctx = r3m.Context(0)
    g = torch.Generator(dev).manual_seed(1)
    spec = torch.randn(r3m.spectral_bytes(n, D, D, r3m.SPEC_C128) // 8, dtype=torch.float64, device=dev, generator=g)
    near = torch.randn((1, n, n), dtype=torch.complex128, device=dev, generator=g)
    store = r3m.Store(n, 2, D, D, 0, r3m.C128, near, r3m.SPEC_C128, spec,
                      common_ext=torch.tensor([0, 1, 2], dtype=torch.int32, device=dev))
    books = [np.random.default_rng(b).integers(0, 2, L * L).astype(np.uint8) for b in range(B)]
    x = torch.randn((B, L * L * 43), dtype=torch.complex128, device=dev, generator=g)

    def product(first, count):
        batch = r3m.Batch.from_codebooks(books[first:first + count], [L] * count, dev)
        xs = x[first:first + count].contiguous()
        work = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, r3m.C128), dtype=torch.uint8, device=dev)
        y = torch.zeros_like(xs)
        r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C128, xs, y, work)
        return y

    y = product(0, B)
    for first in (0, 800, 1579, 1592):  # complex128 products have the same bits at every width
        assert torch.equal(y[first:first + 8], product(first, 8)), first
    ctx.close()
