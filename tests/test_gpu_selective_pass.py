"""The selective second Gram-Schmidt pass (vectors of more than 65,536
entries): every block of a right-hand side acts on one decision, taken before
the pass adds to the coefficients that it depends on, so a solve repeats bit
for bit and converges to its tolerance."""
import numpy as np
import pytest

from workloads import codebooks as cb

import gpu_common as gc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 40 x 41^2 = 67,240 unknowns, beside a short array; nearly equal excitations
# of one codebook pass the criterion at different steps
@pytest.mark.parametrize("refined", [False, True])
def test_long_solves_repeat_bit_for_bit(refined):
    from paper_2112_05082_amd import pipeline, r3m
    dev, L = "cuda:0", 41
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(gc.unit(1), gc.FREQ, 1)
    dense = pipeline.fill_blocks(ctx, geom, L - 1, r3m.C128, dev)
    s64 = pipeline.spectral_store(ctx, geom, L, 2, r3m.C128, dev, dense)
    st = pipeline.spectral_store(ctx, geom, L, 2, r3m.C64, dev, dense) if refined else s64
    sizes = [L, 12]
    batch = r3m.Batch.from_codebooks([cb.bernoulli(n, 3 + n) for n in sizes], sizes, dev, repeat=3)
    N = sum(3 * n * n * 40 for n in sizes)
    b = torch.zeros(N, dtype=torch.complex128, device=dev)
    r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0], [0.3, 0.0, 1.0], [0.9, 0.4, 1.0]] * 2, b)
    work = torch.empty(r3m.gmres_work_bytes(ctx, st, batch, 20, s64 if refined else None,
                                            precond=r3m.PRECOND_BLOCK_JACOBI), dtype=torch.uint8, device=dev)
    tol, runs = 1e-9, []
    for _ in range(4):
        x = torch.zeros_like(b)
        _, rep = r3m.r3m_gmres_solve(ctx, st, s64 if refined else None, batch, b, x, 1e-3 if refined else tol, 20, 4000,
                                     work, refine_tol=tol if refined else 0.0, max_refine=20 if refined else 0,
                                     precond=r3m.PRECOND_BLOCK_JACOBI)
        assert all(r[3] for r in rep)
        runs.append((x, [r[0] for r in rep]))
    for x, iters in runs[1:]:
        assert iters == runs[0][1]
        assert torch.equal(x, runs[0][0])
    y = torch.zeros_like(b)
    mw = torch.empty(r3m.matvec_work_bytes(ctx, s64, batch, r3m.C128), dtype=torch.uint8, device=dev)
    r3m.r3m_retrieved_matvec(ctx, s64, batch, r3m.C128, runs[0][0], y, mw)
    at = 0
    for n in np.repeat(sizes, 3):
        s = slice(at, at + n * n * 40)
        at += n * n * 40
        # the solver's own exit residual is of this product, up to rounding
        assert float((b[s] - y[s]).norm() / b[s].norm()) <= tol * (1 + 1e-3)
    ctx.close()
