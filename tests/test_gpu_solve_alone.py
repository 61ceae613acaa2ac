"""A solve's bits do not depend on what else is in its batch: each right-hand
side takes the Gram-Schmidt form of its own length (the element form above
2,560 unknowns on a complex64 basis, 8,192 on a complex128 one), in batches
with lengths on both sides of these lines, at basis sizes up to and past what
either form folds."""
import numpy as np
import pytest

from workloads import codebooks as cb

import gpu_common as gc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 40 L^2 unknowns: 1,000 (5), 2,560 (8), 3,240 (9), 5,760 (12), 7,840 (14), 9,000
# (15), 16,000 (20), 23,040 (24); GMRES(40) passes the 16 and 32 vectors that the
# forms fold
@pytest.mark.parametrize("sizes,refined,restart", [
    ((12, 24), False, 20), ((14, 15, 3), False, 40), ((8, 9), True, 20), ((8, 14, 20), True, 40), ((5, 15, 8), True, 8)])
def test_batched_solve_equals_each_alone(sizes, refined, restart):
    from paper_2112_05082_amd import pipeline, r3m
    dev, L = "cuda:0", max(sizes)
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(gc.unit(1), gc.FREQ, 1)
    dense = pipeline.fill_blocks(ctx, geom, L - 1, r3m.C128, dev)
    s64 = pipeline.spectral_store(ctx, geom, L, 2, r3m.C128, dev, dense)
    st = pipeline.spectral_store(ctx, geom, L, 2, r3m.C64, dev, dense) if refined else s64
    got = []
    for sel in [list(sizes)] + [[n] for n in sizes]:
        batch = r3m.Batch.from_codebooks([cb.bernoulli(n, 7 + n) for n in sel], sel, dev)
        if refined:  # one frequency product at every width (the matrix-core shapes share their bits)
            r3m.matvec_set_plan(ctx, st, batch, r3m.spec_plan(2, 8))
        b = torch.zeros(sum(n * n * 40 for n in sel), dtype=torch.complex128, device=dev)
        r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[0.3, 0.1, 1.0]] * len(sel), b)
        x = torch.zeros_like(b)
        work = torch.empty(r3m.gmres_work_bytes(ctx, st, batch, restart, s64 if refined else None,
                                                precond=r3m.PRECOND_BLOCK_JACOBI), dtype=torch.uint8, device=dev)
        _, rep = r3m.r3m_gmres_solve(ctx, st, s64 if refined else None, batch, b, x, 1e-3 if refined else 1e-8,
                                     restart, 4000, work, refine_tol=1e-9 if refined else 0.0,
                                     max_refine=20 if refined else 0, precond=r3m.PRECOND_BLOCK_JACOBI)
        assert all(r[3] for r in rep)
        got.append((x.cpu().numpy(), [r[0] for r in rep]))
    assert got[0][1] == [it for _, its in got[1:] for it in its]
    assert np.array_equal(got[0][0], np.concatenate([x for x, _ in got[1:]]))
    ctx.close()
