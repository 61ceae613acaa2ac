"""The streamed frequency product (64 right-hand sides x 80 rows x 8 frequencies
per workgroup, shape {2, 4, 2} of wide batches) against the other matrix-core
kernel: the same sums in the same order, so matvecs and solves agree bit for
bit, over whole and ragged tiles of rows and right-hand sides, one to many
tiles per workgroup, and a live list that shrinks during a solve.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_common import FREQ, unit  # noqa: E402
from workloads import codebooks as cb  # noqa: E402

DEV = "cuda:0"


# n = n_a S: 64, 80, 160, 192, 256 rows (row groups of 80: whole, and with one
# and two 16-row tiles); transform grids 4 x 4, 16 x 16, 64 x 64 (2 to 512
# frequency tiles); the last 64 right-hand sides: 1, 49, 64
@pytest.mark.parametrize("n_a,S,D,B", [(40, 2, 1, 49), (40, 2, 7, 64), (40, 4, 7, 65), (64, 1, 7, 64), (64, 3, 1, 113),
                                       (64, 4, 1, 128), (40, 2, 24, 128), (40, 2, 24, 193)])
def test_product_stream_bits(n_a, S, D, B):
    from paper_2112_05082_amd import r3m
    ctx = r3m.Context(0)
    n, L = n_a * S, D + 1
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


def test_solve_identical_with_stream():
    """80 right-hand sides at 8 x 8, one tile of 16 idle from the start."""
    from paper_2112_05082_amd import pipeline, r3m
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit(1), FREQ, 1)
    L, n_books, angles = 8, 20, (0.0, 20.0, 40.0, 60.0)
    books = [cb.family(c % 3, L, 7300 + c) for c in range(n_books)]
    batch = r3m.Batch.from_codebooks(books, [L] * n_books, DEV, repeat=len(angles))
    n1 = L * L * 40
    spec = pipeline.spectral_store(ctx, geom, L, 2, r3m.C64, DEV)
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


@pytest.mark.parametrize("n_a,S,D", [(40, 2, 1), (40, 2, 11), (64, 3, 3)])
def test_c128_product_two_tiles(n_a, S, D):
    """Complex128 products of more than 16 right-hand sides (two tiles per
    workgroup: 17 and 32, then 33 and 130 with an unpaired and a ragged last
    tile) equal those of 5 at a time bit for bit."""
    from paper_2112_05082_amd import r3m
    ctx = r3m.Context(0)
    n, L = n_a * S, D + 1
    g = torch.Generator(DEV).manual_seed(D)
    spec = torch.randn(r3m.spectral_bytes(n, D, D, r3m.SPEC_C128) // 8, dtype=torch.float64, device=DEV, generator=g)
    near = torch.randn((1, n, n), dtype=torch.complex128, device=DEV, generator=g)
    store = r3m.Store(n, S, D, D, 0, r3m.C128, near, r3m.SPEC_C128, spec)
    books = [np.random.default_rng(b).integers(0, S, L * L).astype(np.uint8) for b in range(130)]
    x = torch.randn((130, L * L * n_a), dtype=torch.complex128, device=DEV, generator=g)

    def product(first, count):
        batch = r3m.Batch.from_codebooks(books[first:first + count], [L] * count, DEV)
        xs = x[first:first + count].contiguous()
        work = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, r3m.C128), dtype=torch.uint8, device=DEV)
        y = torch.zeros_like(xs)
        r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C128, xs, y, work)
        return y

    ref = torch.cat([product(i, 5) for i in range(0, 130, 5)])
    for count in (17, 32, 33, 130):
        assert torch.equal(product(0, count), ref[:count])
    ctx.close()
