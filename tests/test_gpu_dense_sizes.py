"""Dense products past the one-launch kernel's lines, every value against the
sum over unit pairs: the lists and the slab kernel for 40 bases a state, and
states of 64, which the slab kernel does not take at any size."""
import numpy as np
import pytest

from test_gpu_dense_direct import case, product

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 64 bases: 169 units alone, 153,664 pairs, arrays of one row; 40 bases: the
# lists from 28,672 or 32,768 pairs, the slab kernel from 28,672, 40,960 or
# 131,072 (by type, states and how well its 8x8 tiles fit the array)
@pytest.mark.parametrize("n_a,S,D,shapes", [
    (64, 1, 12, [(13, 13)]), (64, 2, 13, [(14, 14)] * 4), (64, 2, 19, [(20, 8), (1, 20), (13, 13)]),
    (64, 2, 5, [(6, 6)] * 26), (40, 2, 5, [(6, 6)] * 26), (40, 1, 13, [(14, 14)] * 4),
    (40, 2, 5, [(6, 6)] * 23), (40, 4, 4, [(5, 5)] * 48), (40, 4, 3, [(4, 4)] * 120), (40, 2, 3, [(4, 4)] * 120),
    (40, 1, 13, [(14, 14)]), (40, 2, 14, [(15, 15)]), (40, 2, 7, [(8, 8)] * 33), (40, 1, 7, [(7, 7)] * 56),
    (40, 2, 23, [(24, 2), (15, 15)])])
@pytest.mark.parametrize("store,vec", [("c128", "c128"), ("c64", "c128"), ("c64", "c64")])
def test_dense_product(n_a, S, D, shapes, store, vec):
    from paper_2112_05082_amd import r3m
    rng = np.random.default_rng(D + 100 * S)
    n, Z, uoff, soff, states, x = case(rng, n_a, S, D, shapes)
    dev, code, tdt = "cuda:0", {"c128": r3m.C128, "c64": r3m.C64}, {"c128": torch.complex128, "c64": torch.complex64}
    ctx = r3m.Context(0)
    st = r3m.Store(n, S, D, D, D, code[store], torch.from_numpy(Z).to(dev).to(tdt[store]))
    batch = r3m.Batch(shapes, uoff, soff, torch.from_numpy(states).to(dev))
    xd = torch.from_numpy(x).to(dev).to(tdt[vec])
    y = torch.zeros_like(xd)
    work = torch.empty(r3m.matvec_work_bytes(ctx, st, batch, code[vec]), dtype=torch.uint8, device=dev)
    r3m.r3m_retrieved_matvec(ctx, st, batch, code[vec], xd, y, work)
    r3m.r3m_ctx_check(ctx)
    # sums of n_a units products: rounding of their number's root, FP64 (1e-13)
    # or FP32 (1e-5) of the largest
    ref = product(Z, n_a, D, shapes, uoff, soff, states, x)
    assert np.abs(y.cpu().numpy() - ref).max() <= (1e-13 if store == "c128" else 1e-5) * np.abs(ref).max()
    ctx.close()
