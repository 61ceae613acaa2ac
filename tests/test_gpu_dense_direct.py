"""The one-launch dense product at the edges of its rule: pair counts on both
sides of it, 40 and 64 bases a state, one to four states, ragged batches with
gaps between the vectors, vectors in place, and the state check."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def case(rng, n_a, S, D, shapes):
    n = n_a * S
    Z = rng.standard_normal(((2 * D + 1) ** 2, n, n)) + 1j * rng.standard_normal(((2 * D + 1) ** 2, n, n))
    uoff, soff, u, s = [], [], 3, 0
    for Lx, Ly in shapes:
        uoff.append(u)
        soff.append(s)
        u += Lx * Ly + 2  # gaps between the vectors
        s += Lx * Ly
    states = rng.integers(0, S, s).astype(np.uint8)
    x = rng.standard_normal((u * n_a)) + 1j * rng.standard_normal(u * n_a)
    return n, Z, uoff, soff, states, x


def product(Z, n_a, D, shapes, uoff, soff, states, x):
    y = np.zeros_like(x)
    for (Lx, Ly), uo, so in zip(shapes, uoff, soff):
        xb = x[uo * n_a:(uo + Lx * Ly) * n_a].reshape(-1, n_a)
        for i in range(Lx * Ly):
            for j in range(Lx * Ly):
                d = (i // Lx - j // Lx + D) * (2 * D + 1) + i % Lx - j % Lx + D
                a, b = states[so + i] * n_a, states[so + j] * n_a
                y[(uo + i) * n_a:(uo + i + 1) * n_a] += Z[d, a:a + n_a, b:b + n_a] @ xb[j]
    return y


# the last two lie past the rule (32,768 pairs against the lists; more than 144
# units and 131,072 pairs against the slab kernel)
@pytest.mark.parametrize("n_a,S,D,shapes", [
    (40, 2, 0, [(1, 1)]), (40, 1, 2, [(3, 3), (1, 2)]), (40, 4, 3, [(4, 4), (3, 1), (2, 4)]), (64, 2, 4, [(5, 5), (5, 2)]),
    (40, 2, 7, [(8, 8), (7, 3)]), (40, 2, 11, [(12, 12)]), (40, 2, 5, [(6, 6)] * 26), (40, 1, 13, [(14, 14)] * 4)])
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
    y = torch.full_like(xd, 7.0)
    work = torch.empty(r3m.matvec_work_bytes(ctx, st, batch, code[vec]), dtype=torch.uint8, device=dev)
    r3m.r3m_retrieved_matvec(ctx, st, batch, code[vec], xd, y, work)
    r3m.r3m_ctx_check(ctx)
    got = y.cpu().numpy()
    used = np.zeros(len(x), bool)
    for (Lx, Ly), uo in zip(shapes, uoff):
        used[uo * n_a:(uo + Lx * Ly) * n_a] = True
    assert np.all(got[~used] == 7.0)  # nothing outside the vectors is written
    if sum((a * b) ** 2 for a, b in shapes) <= 20000 or len(shapes) == 1:
        ref = product(Z, n_a, D, shapes, uoff, soff, states, x)
        # sums of n_a units products: rounding of their number's root, FP64
        # (1e-13) or FP32 (1e-5) of the largest
        tol = 1e-13 if store == "c128" else 1e-5
        assert np.abs(got[used] - ref[used]).max() <= tol * np.abs(ref).max()
    r3m.r3m_retrieved_matvec(ctx, st, batch, code[vec], xd, xd, work)  # in place
    assert np.array_equal(xd.cpu().numpy()[used], got[used])
    ctx.close()


def test_bad_state_is_reported():
    from paper_2112_05082_amd import r3m
    dev = "cuda:0"
    ctx = r3m.Context(0)
    st = r3m.Store(80, 2, 1, 1, 1, r3m.C128, torch.ones((9, 80, 80), dtype=torch.complex128, device=dev))
    states = torch.tensor([0, 1, 2, 0], dtype=torch.uint8, device=dev)
    batch = r3m.Batch([(2, 2)], [0], [0], states)
    x = torch.ones(160, dtype=torch.complex128, device=dev)
    y = torch.zeros_like(x)
    work = torch.empty(r3m.matvec_work_bytes(ctx, st, batch, r3m.C128), dtype=torch.uint8, device=dev)
    r3m.r3m_retrieved_matvec(ctx, st, batch, r3m.C128, x, y, work)
    with pytest.raises(r3m.R3MError):
        r3m.r3m_ctx_check(ctx)
    r3m.r3m_ctx_check(ctx)  # cleared
    ctx.close()


@pytest.mark.parametrize("L", [3, 8, 17])
def test_bad_state_is_reported_by_the_lists(L):
    """Compressed stores check the states while they build their lists."""
    from paper_2112_05082_amd import pipeline, r3m
    from gpu_common import FREQ, unit
    dev = "cuda:0"
    ctx = r3m.Context(0)
    geom = r3m.UnitGeom.from_macro(unit(1), FREQ, 1)
    st = pipeline.compressed_store(ctx, geom, L, 1, r3m.C64, r3m.C64, 1e-3, 12, dev)
    states = torch.zeros(2 * L * L, dtype=torch.uint8, device=dev)
    batch = r3m.Batch([(L, L), (L, L)], [0, L * L], [0, L * L], states)
    x = torch.ones(2 * L * L * 40, dtype=torch.complex64, device=dev)
    y = torch.zeros_like(x)
    work = torch.empty(r3m.matvec_work_bytes(ctx, st, batch, r3m.C64), dtype=torch.uint8, device=dev)
    for at, bad in ((None, False), (2 * L * L - 1, True), (0, True)):
        states.zero_()
        if at is not None:
            states[at] = 2
        r3m.r3m_retrieved_matvec(ctx, st, batch, r3m.C64, x, y, work)
        if bad:
            with pytest.raises(r3m.R3MError):
                r3m.r3m_ctx_check(ctx)
        r3m.r3m_ctx_check(ctx)
    assert r3m.matvec_groups(ctx, st, batch) >= 1
    ctx.close()
