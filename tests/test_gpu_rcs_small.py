"""RCS of arrays of at most 256 units, whose passes the waves take in turn: unit
counts on both sides of that line in one batch, fewer passes than waves and
more, shared bases, and several chunks whose last is small."""
import numpy as np
import pytest

from gpu_common import FREQ, K
from oracle import efie, farfield
from workloads import codebooks as cb
from workloads.mesh import macro_unit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# bases a state 1, 40, 65: passes of 40 entries, n_states (1 or 2) of them;
# (33, 8): 1,089 units in chunks of 1,024, the last of 65
@pytest.mark.parametrize("ncell,S,sizes,n_dir", [
    (4, 1, (16, 17, 1), 33), (4, 2, (16, 17, 15), 16), (4, 4, (16, 17, 6), 40), (5, 3, (2, 16), 18),
    (1, 7, (16, 17), 5), (4, 2, (33, 8), 32)])
def test_rcs_of_small_arrays(ncell, S, sizes, n_dir):
    from paper_2112_05082_amd import r3m
    unit = macro_unit(tuple(np.linspace(0.005, 0.011, S)), ncell)
    ctx, dev = r3m.Context(0), "cuda:0"
    geom = r3m.UnitGeom.from_macro(unit, FREQ, 1)
    books = [cb.uniform(L, S, 5 + L) for L in sizes]
    books[0][:] = S - 1  # one state only: the other passes are empty
    batch = r3m.Batch.from_codebooks(books, list(sizes), dev)
    I = cb.random_complex(sum(L * L for L in sizes) * unit.n_a, 3)
    rng = np.random.default_rng(5)
    dirs = np.stack([rng.uniform(-np.pi, np.pi, n_dir), rng.uniform(0, 2 * np.pi, n_dir)], 1)
    sigma = torch.full((len(sizes) * n_dir,), float("nan"), dtype=torch.float64, device=dev)
    r3m.r3m_rcs(ctx, geom, batch, torch.from_numpy(I).to(dev), dirs, 2.0, sigma)
    sigma = sigma.cpu().numpy().reshape(len(sizes), n_dir)
    at = 0
    for i, L in enumerate(sizes):
        mesh, _ = efie.active_array_mesh(unit, books[i], L)
        n = L * L * unit.n_a
        ref = farfield.rcs(mesh, I[at:at + n], K, dirs, 2.0)
        # phases k r below 300 rounded to 2^-53 of themselves (3e-14) in sums
        # whose terms have no common phase, squared: 1e-11
        assert np.abs(sigma[i] - ref).max() <= 1e-11 * ref.max()
        at += n
    ctx.close()
