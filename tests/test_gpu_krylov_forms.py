"""Gram-Schmidt forms of the solver: vector lengths on both sides of the lines
between the split and the element-parallel update and between coefficients
summed in the update and in a launch of their own, alone and in ragged batches."""
import numpy as np
import pytest

from workloads import codebooks as cb

import gpu_common as gc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 40 L^2 unknowns: 320 and 1,000 (few partials, added one by one), 7,840 and
# 9,000 (the complex64 line at 8,192), 16,000 and 17,640 (the complex128 one
# at 16,384), 67,240 (past 64 chunks); the folded update's 128 partials lie at
# 8,192 and 32,768
@pytest.mark.parametrize("sizes", [(2, 3), (5,), (14,), (15, 9), (20,), (21, 4), (30, 13), (41,)])
@pytest.mark.parametrize("refined", [False, True])
def test_solve_forms(sizes, refined):
    from paper_2112_05082_amd import pipeline, r3m
    dev, L = "cuda:0", max(sizes)
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(gc.unit(1), gc.FREQ, 1)
    dense = pipeline.fill_blocks(ctx, geom, L - 1, r3m.C128, dev)
    s64 = pipeline.spectral_store(ctx, geom, L, 2, r3m.C128, dev, dense)
    st = pipeline.spectral_store(ctx, geom, L, 2, r3m.C64, dev, dense) if refined else s64
    batch = r3m.Batch.from_codebooks([cb.bernoulli(n, 7 + n) for n in sizes], list(sizes), dev, repeat=2)
    N = sum(2 * n * n * 40 for n in sizes)
    b = torch.zeros(N, dtype=torch.complex128, device=dev)
    r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0], [0.5, 0.0, 1.0]] * len(sizes), b)
    x, y = torch.zeros_like(b), torch.zeros_like(b)
    wb = r3m.gmres_work_bytes(ctx, st, batch, 20, s64 if refined else None, precond=r3m.PRECOND_BLOCK_JACOBI)
    work = torch.empty(wb, dtype=torch.uint8, device=dev)
    tol = 1e-9
    _, rep = r3m.r3m_gmres_solve(ctx, st, s64 if refined else None, batch, b, x, 1e-3 if refined else tol, 20, 4000,
                                 work, refine_tol=tol if refined else 0.0, max_refine=20 if refined else 0,
                                 precond=r3m.PRECOND_BLOCK_JACOBI)
    mw = torch.empty(r3m.matvec_work_bytes(ctx, s64, batch, r3m.C128), dtype=torch.uint8, device=dev)
    r3m.r3m_retrieved_matvec(ctx, s64, batch, r3m.C128, x, y, mw)
    at = 0
    for i, n in enumerate(n for n in sizes for _ in range(2)):
        s = slice(at, at + n * n * 40)
        at += n * n * 40
        assert rep[i][3]
        # the solver's own exit residual is of this product, up to rounding
        assert float((b[s] - y[s]).norm() / b[s].norm()) <= tol * (1 + 1e-3)
    ctx.close()


@pytest.mark.parametrize("L", [9, 15])
def test_small_vector_independent_of_width(L):
    """Up to the first line a batch of equal arrays solves as each alone, bit for bit."""
    from paper_2112_05082_amd import pipeline, r3m
    dev = "cuda:0"
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(gc.unit(1), gc.FREQ, 1)
    st = pipeline.spectral_store(ctx, geom, L, 2, r3m.C128, dev)
    books = [cb.bernoulli(L, k) for k in range(3)]
    got = []
    for sel in ([0, 1, 2], [1]):
        batch = r3m.Batch.from_codebooks([books[k] for k in sel], [L] * len(sel), dev)
        b = torch.zeros(len(sel) * L * L * 40, dtype=torch.complex128, device=dev)
        r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.0, 0.0, 1.0]] * len(sel), b)
        x = torch.zeros_like(b)
        work = torch.empty(r3m.gmres_work_bytes(ctx, st, batch, 20, precond=r3m.PRECOND_BLOCK_JACOBI),
                           dtype=torch.uint8, device=dev)
        r3m.r3m_gmres_solve(ctx, st, None, batch, b, x, 1e-8, 20, 2000, work, precond=r3m.PRECOND_BLOCK_JACOBI)
        got.append(x.cpu().numpy())
    n = L * L * 40
    assert np.array_equal(got[0][n:2 * n], got[1])
    ctx.close()
