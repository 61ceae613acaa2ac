"""RCS and excitation at the edges of their tiles: directions around 16 and 32,
entries around a pass of 40 (1, 40, 65 bases a state), unit counts around a
list of 256 and a chunk of 1,024, states that are missing from a list."""
import numpy as np
import pytest

from gpu_common import FREQ, K
from oracle import efie, excitation, farfield
from workloads import codebooks as cb
from workloads.mesh import macro_unit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncell,sides,sizes,n_dir", [
    (4, (0.006, 0.009), (1, 2), 1), (4, (0.006, 0.009), (16, 17), 16), (4, (0.006,), (15,), 33),
    (1, (0.006, 0.009), (33, 3), 17), (5, (0.006, 0.009), (5, 4), 31), (4, (0.005, 0.007, 0.009, 0.011), (6, 32), 32),
    # more than 2,048 workgroups: a chunk of 2,048 units
    (1, (0.006, 0.009), (33, 40) + (1,) * 60, 600)])
def test_rcs_and_excitation(ncell, sides, sizes, n_dir):
    from paper_2112_05082_amd import r3m
    unit = macro_unit(sides, ncell)
    dev = "cuda:0"
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit, FREQ, 1)
    books = [cb.uniform(L, len(sides), 11 + L) for L in sizes]
    books[0][: len(books[0]) // 2] = 0  # the first list has one state only
    batch = r3m.Batch.from_codebooks(books, list(sizes), dev)
    N = sum(L * L for L in sizes) * unit.n_a
    I = cb.random_complex(N, 3)
    rng = np.random.default_rng(5)
    dirs = np.stack([rng.uniform(-np.pi, np.pi, n_dir), rng.uniform(0, 2 * np.pi, n_dir)], 1)
    inc = [[0.3 + 0.2 * i, 1.1 * i, 1.0 + i] for i in range(len(sizes))]
    b = torch.full((N,), float("nan"), dtype=torch.complex128, device=dev)
    sigma = torch.full((len(sizes) * n_dir,), float("nan"), dtype=torch.float64, device=dev)
    r3m.r3m_plane_wave_rhs(ctx, geom, batch, inc, b)
    r3m.r3m_rcs(ctx, geom, batch, torch.from_numpy(I).to(dev), dirs, 2.0, sigma)
    b, sigma = b.cpu().numpy(), sigma.cpu().numpy().reshape(len(sizes), n_dir)
    at = 0
    for i, L in enumerate(sizes):
        mesh, _ = efie.active_array_mesh(unit, books[i], L)
        n = L * L * unit.n_a
        # phases k r below 300 rounded to 2^-53 of themselves (3e-14), a few
        # of them per term: 1e-12 of the largest value; sigma is quadratic in
        # sums whose terms have no common phase: 1e-11
        U = excitation.plane_wave(mesh, K, *inc[i])
        assert np.abs(b[at:at + n] - U).max() <= 1e-12 * np.abs(U).max()
        ref = farfield.rcs(mesh, I[at:at + n], K, dirs, 2.0)
        assert np.abs(sigma[i] - ref).max() <= 1e-11 * ref.max()
        at += n
    ctx.close()
