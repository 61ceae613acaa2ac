"""Line transforms at every stage pattern: transform lengths 2 to 512 (one
stage, two, a remainder of radix 2, 4 or 8, three), square and not, block
sizes with one grid or several to a workgroup, against numpy's FFT."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 2 D + 1 <= G: D = 0, 1, 3, 7, 15, 31, 63, 127, 255 give G = 2 to 512
@pytest.mark.parametrize("n,Dx,Dy", [(1, 0, 0), (3, 0, 1), (4, 1, 3), (12, 3, 2), (80, 7, 7), (5, 15, 7), (16, 15, 31),
                                     (7, 31, 20), (4, 63, 5), (3, 2, 127), (2, 255, 40), (24, 8, 33)])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_spectra_of_random_blocks(n, Dx, Dy, dtype):
    from paper_2112_05082_amd import r3m
    ctx = r3m.Context(0)
    c64 = dtype == "c64"
    sd = r3m.SPEC_C64 if c64 else r3m.SPEC_C128
    rng = np.random.default_rng(n + 10 * Dx + 1000 * Dy)
    Sx, Sy = 2 * Dx + 1, 2 * Dy + 1
    Z = rng.standard_normal((Sy, Sx, n, n)) + 1j * rng.standard_normal((Sy, Sx, n, n))
    Gx, Gy = (max(2, 1 << (S - 1).bit_length()) for S in (Sx, Sy))
    out = torch.full((n, n, Gy, Gx), float("nan"), dtype=torch.complex64 if c64 else torch.complex128, device="cuda:0")
    assert r3m.spectral_bytes(n, Dx, Dy, sd) == out.numel() * out.element_size()
    r3m.r3m_build_spectral(ctx, torch.from_numpy(Z).to("cuda:0"), n, Dx, Dy, sd, out)
    E = np.zeros((Gy, Gx, n, n), complex)
    E[np.ix_(np.arange(-Dy, Dy + 1) % Gy, np.arange(-Dx, Dx + 1) % Gx)] = Z
    ref = np.fft.fft2(E, axes=(0, 1)).transpose(2, 3, 0, 1)
    # log2(Gx Gy) butterflies, each adding a few units of rounding to values
    # of the size of the root mean square: 1e-6 (float) and 3e-15 (double) of
    # the largest
    assert np.abs(out.cpu().numpy() - ref).max() <= (1e-6 if c64 else 3e-15) * np.abs(ref).max()
    ctx.close()


@pytest.mark.parametrize("L,D", [(1, 0), (2, 1), (3, 4), (5, 9), (9, 17), (11, 33), (6, 70)])
def test_matvec_two_pass_lengths(L, D):
    """Products through the masked passes on small and on oversized grids,
    complex128 against the dense product, complex64 fused against two passes."""
    from paper_2112_05082_amd import r3m
    dev, n = "cuda:0", 80
    ctx = r3m.Context(0)
    rng = np.random.default_rng(L + D)
    S = 2 * D + 1
    Z = torch.zeros((S, S, n, n), dtype=torch.complex128)
    a, b = D - L + 1, D + L
    Z[a:b, a:b] = torch.from_numpy(rng.standard_normal((2 * L - 1, 2 * L - 1, n, n)) +
                                   1j * rng.standard_normal((2 * L - 1, 2 * L - 1, n, n)))
    Zd = Z.view(S * S, n, n).to(dev)
    states = rng.integers(0, 2, L * L).astype(np.uint8)
    batch = r3m.Batch([(L, L), (L, 1)], [0, L * L], [0, 0], torch.from_numpy(states).to(dev))
    x = rng.standard_normal((L * L + L) * 40) + 1j * rng.standard_normal((L * L + L) * 40)
    got = {}
    for name, sd, vt, tdt in (("c128", r3m.SPEC_C128, r3m.C128, torch.complex128),
                              ("c64", r3m.SPEC_C64, r3m.C64, torch.complex64)):
        spec = torch.empty(r3m.spectral_bytes(n, D, D, sd), dtype=torch.uint8, device=dev)
        r3m.r3m_build_spectral(ctx, Zd, n, D, D, sd, spec)
        store = r3m.Store(n, 2, D, D, 0, vt, Zd.view(S, S, n, n)[D, D][None].to(tdt).contiguous(), sd, spec)
        work = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, vt), dtype=torch.uint8, device=dev)
        xd = torch.from_numpy(x).to(dev).to(tdt)
        for two in ((False,) if name == "c128" else (False, True)):
            if name == "c64":
                r3m.matvec_set_plan(ctx, store, batch, r3m.spec_plan(0, two_pass=two))
            y = torch.full_like(xd, float("nan"))
            r3m.r3m_retrieved_matvec(ctx, store, batch, vt, xd, y, work)
            got[name, two] = y.cpu().numpy()
    Zn, ref, at = Z.numpy(), [], 0
    for Lx, Ly in ((L, L), (L, 1)):
        xb = x[at:at + Lx * Ly * 40].reshape(Ly * Lx, 40)
        at += Lx * Ly * 40
        for i in range(Lx * Ly):
            acc = np.zeros(40, complex)
            for j in range(Lx * Ly):
                blk = Zn[i // Lx - j // Lx + D, i % Lx - j % Lx + D]
                si, sj = states[i] * 40, states[j] * 40
                acc += blk[si:si + 40, sj:sj + 40] @ xb[j]
            ref.append(acc)
    ref = np.concatenate(ref)
    # products of 40 L^2 random terms: rounding of the transforms and sums, a
    # few units each, relative to the root of their number
    assert np.abs(got["c128", False] - ref).max() <= 1e-13 * np.abs(ref).max()
    assert np.abs(got["c64", False] - ref).max() <= 5e-6 * np.abs(ref).max()
    assert np.array_equal(got["c64", False], got["c64", True])
    ctx.close()


@pytest.mark.parametrize("n_a,S,L,common", [(40, 2, 3, 0), (40, 4, 5, 0), (64, 1, 9, 0), (40, 2, 17, 3), (40, 4, 33, 0)])
def test_c128_product_independent_of_width(n_a, S, L, common):
    """One and two right-hand sides run on the vector units, more on the matrix
    cores: the same bits, forward and (isolated units) transposed."""
    from paper_2112_05082_amd import r3m
    dev, n, D = "cuda:0", n_a * S + common, L - 1
    ctx = r3m.Context(0)
    g = torch.Generator(dev).manual_seed(L)
    spec = torch.randn(r3m.spectral_bytes(n, D, D, r3m.SPEC_C128) // 8, dtype=torch.float64, device=dev, generator=g)
    near = torch.randn((1, n, n), dtype=torch.complex128, device=dev, generator=g)
    ext = torch.arange(common, dtype=torch.int32, device=dev) % 3 if common else None
    store = r3m.Store(n, S, D, D, 0, r3m.C128, near, r3m.SPEC_C128, spec, common_ext=ext)
    per = n_a + common
    rng = np.random.default_rng(L)
    books = [rng.integers(0, S, L * L).astype(np.uint8) for _ in range(5)]
    x = torch.randn(5 * L * L * per, dtype=torch.complex128, device=dev, generator=g)
    w = torch.rand((5 * L * L, S), dtype=torch.float64, device=dev, generator=g)
    ref = {}
    for width in (5, 1, 2):
        for first in range(0, 5 - width + 1, 2):
            ids = list(range(first, first + width))
            batch = r3m.Batch.from_codebooks([books[i] for i in ids], [L] * width, dev)
            xs = x[first * L * L * per:(first + width) * L * L * per].contiguous()
            work = torch.empty(r3m.matvec_work_bytes(ctx, store, batch, r3m.C128), dtype=torch.uint8, device=dev)
            out = [torch.zeros_like(xs)]
            r3m.r3m_retrieved_matvec(ctx, store, batch, r3m.C128, xs, out[0], work)
            if not common:
                ws = w[first * L * L:(first + width) * L * L].contiguous()
                work = torch.empty(r3m.relaxed_work_bytes(ctx, store, batch), dtype=torch.uint8, device=dev)
                for tr in (False, True):
                    out.append(torch.zeros_like(xs))
                    r3m.r3m_relaxed_matvec(ctx, store, batch, ws, r3m.C128, xs, out[-1], work, transpose=tr)
            for k, y in enumerate(out):
                y = y.cpu().numpy().reshape(width, -1)
                for i, row in zip(ids, y):
                    if width == 5:
                        ref[k, i] = row
                    else:
                        assert np.array_equal(row, ref[k, i])
    ctx.close()
