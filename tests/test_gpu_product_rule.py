"""The streamed frequency product on the batches that its rule gives it (129 to
256 items of 8 frequencies x 80 rows x 64 right-hand sides, or more than 384)
against the other matrix-core kernel, bit for bit: row groups that end after
one, two or four 16-row tiles, ragged right-hand sides, few frequencies with
many right-hand sides, and a live list that shrinks during a solve."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_common import FREQ, unit  # noqa: E402
from workloads import codebooks as cb  # noqa: E402

DEV = "cuda:0"


# 64 x 64 grids with n = 64, 192, 256; 32 x 32 ones with 80, 160; 16 x 16 and
# 4 x 4 ones
@pytest.mark.parametrize("n_a,S,D,B", [(64, 1, 24, 49), (64, 3, 24, 64), (64, 4, 24, 113), (40, 4, 15, 65),
                                       (40, 2, 15, 100), (40, 2, 7, 300), (40, 2, 1, 4200), (40, 2, 31, 66)])
def test_product_bits(n_a, S, D, B):
    from paper_2112_05082_amd import r3m
    ctx = r3m.Context(0)
    n, L = n_a * S, min(D + 1, 4)
    g = torch.Generator(DEV).manual_seed(B)
    spec = torch.randn(r3m.spectral_bytes(n, D, D, r3m.SPEC_C64) // 4, dtype=torch.float32, device=DEV, generator=g)
    near = torch.randn((1, n, n), dtype=torch.complex64, device=DEV, generator=g)
    store = r3m.Store(n, S, D, D, 0, r3m.C64, near, r3m.SPEC_C64, spec)
    books = [np.random.default_rng(b).integers(0, S, L * L).astype(np.uint8) for b in range(B)]
    batch = r3m.Batch.from_codebooks(books, [L] * B, DEV)
    x = torch.randn(B * L * L * n_a, dtype=torch.complex64, device=DEV, generator=g)
    work = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, r3m.C64), dtype=torch.uint8, device=DEV)
    out = []
    for shape in (2, 6):
        r3m.matvec_set_plan(ctx, store, batch, r3m.spec_plan(shape, 8))
        y = torch.zeros_like(x)
        r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C64, x, y, work)
        out.append(y)
    assert torch.equal(*out)
    ctx.close()


def test_solve_with_shrinking_list():
    """64 right-hand sides at 8 x 8 on a store for 32 x 32, one tile of 16 idle
    from the start."""
    from paper_2112_05082_amd import pipeline, r3m
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit(1), FREQ, 1)
    L, n_books, angles = 8, 16, (0.0, 20.0, 40.0, 60.0)
    books = [cb.family(c % 3, L, 7300 + c) for c in range(n_books)]
    batch = r3m.Batch.from_codebooks(books, [L] * n_books, DEV, repeat=len(angles))
    n1 = L * L * 40
    spec = pipeline.spectral_store(ctx, geom, 32, 2, r3m.C64, DEV)
    b = torch.zeros(batch.B * n1, dtype=torch.complex128, device=DEV)
    r3m.r3m_plane_wave_rhs(ctx, geom, batch, [[np.deg2rad(a), 0.0, 1.0] for _ in range(n_books) for a in angles], b)
    b[16 * n1:32 * n1] = 0
    work = torch.empty(r3m.gmres_work_bytes(ctx, spec, batch, 8), dtype=torch.uint8, device=DEV)
    out = []
    for shape in (2, 6):
        r3m.matvec_set_plan(ctx, spec, batch, r3m.spec_plan(shape, 8))
        x = torch.zeros_like(b)
        rc, rep = r3m.r3m_gmres_solve(ctx, spec, None, batch, b, x, 1e-5, 8, 4000, work,
                                      precond=r3m.PRECOND_BLOCK_JACOBI)
        assert rc == 0 and all(r[3] for r in rep)
        out.append((x, [r[0] for r in rep]))
    assert len(set(out[0][1])) >= 4 and out[0][1] == out[1][1]
    assert torch.equal(out[0][0], out[1][0])
    ctx.close()


def test_tuned_plan_of_a_streamed_batch():
    """The streamed kernel has one workgroup order: the tuner does not choose
    between two of them, and pinned order bits change nothing."""
    from paper_2112_05082_amd import r3m
    ctx = r3m.Context(0)
    n, D, B, L = 80, 31, 128, 4
    g = torch.Generator(DEV).manual_seed(B)
    spec = torch.randn(r3m.spectral_bytes(n, D, D, r3m.SPEC_C64) // 4, dtype=torch.float32, device=DEV, generator=g)
    near = torch.randn((1, n, n), dtype=torch.complex64, device=DEV, generator=g)
    store = r3m.Store(n, 2, D, D, 0, r3m.C64, near, r3m.SPEC_C64, spec)
    books = [np.random.default_rng(b).integers(0, 2, L * L).astype(np.uint8) for b in range(B)]
    x = torch.randn(B * L * L * 40, dtype=torch.complex64, device=DEV, generator=g)
    out = []
    for plan in (None, r3m.spec_plan(6, 64), r3m.spec_plan(6, 1), r3m.spec_plan(6, 255, kt_groups=2)):
        batch = r3m.Batch.from_codebooks(books, [L] * B, DEV)
        if plan is not None:
            r3m.matvec_set_plan(ctx, store, batch, plan)
        work = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, r3m.C64), dtype=torch.uint8, device=DEV)
        y = torch.zeros_like(x)
        r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C64, x, y, work)
        got = r3m.matvec_plan(ctx, store, batch)
        if plan is None and got & 15 == 6:
            assert (got >> 4) & 255 == 64
        if plan is not None:
            assert got == plan
            out.append(y)
    assert all(torch.equal(y, out[0]) for y in out[1:])
    ctx.close()
