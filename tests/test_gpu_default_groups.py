"""The untuned displacement-group count weighs the workgroups' rounds against
the partial sums that every group adds, and the product does not depend on it
beyond rounding order."""
import numpy as np
import pytest

from workloads import codebooks as cb

from gpu_common import FREQ, unit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# one tile an array: 8 x 96 workgroups would fill the chip, but 169
# displacements are too few to split that far (us at 64, 96 groups: 33, 36)
@pytest.mark.parametrize("L,B,low,high", [(6, 8, 32, 80), (8, 6, 48, 96), (8, 1, 64, 128), (16, 6, 24, 48)])
def test_default_groups(L, B, low, high):
    from paper_2112_05082_amd import pipeline, r3m
    dev = "cuda:0"
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit(1), FREQ, 1)
    st = pipeline.compressed_store(ctx, geom, L, 1, r3m.C64, r3m.C64, 1e-3, 12, dev)
    batch = r3m.Batch.from_codebooks([cb.bernoulli(L, k) for k in range(B)], [L] * B, dev)
    g = r3m.matvec_groups(ctx, st, batch)
    assert low <= g <= high
    x = torch.randn(B * L * L * 40, dtype=torch.complex64, device=dev, generator=torch.Generator(dev).manual_seed(1))
    work = torch.empty(r3m.matvec_work_bytes(ctx, st, batch, r3m.C64), dtype=torch.uint8, device=dev)
    got = []
    for k in (None, 1, 7):
        if k:
            r3m.matvec_set_plan(ctx, st, batch, k)
        y = torch.zeros_like(x)
        r3m.r3m_retrieved_matvec(ctx, st, batch, r3m.C64, x, y, work)
        got.append(y.cpu().numpy())
    # sums of 40 L^2 products in FP32, rounded in another order
    for y in got[1:]:
        assert np.abs(y - got[0]).max() <= 1e-5 * np.abs(got[0]).max()
    ctx.close()
