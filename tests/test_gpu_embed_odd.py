"""Block spectra of unit sizes that no power of two divides: the last workgroup
of a row has lines to spare, and the build costs what its neighbours' do."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# n^2 grids in groups of 4096 / G (complex64) or 2048 / G lines: 81 in groups
# of 64 and 32, 121 of 16 and 8, 9 in one group, 225 of 256 and 128, 25 of 2048
@pytest.mark.parametrize("n,Dx,Dy", [(9, 31, 3), (11, 127, 2), (3, 15, 0), (15, 7, 5), (5, 0, 9), (6, 31, 2)])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_spectra_of_odd_units(n, Dx, Dy, dtype):
    from paper_2112_05082_amd import r3m
    ctx = r3m.Context(0)
    c64 = dtype == "c64"
    sd = r3m.SPEC_C64 if c64 else r3m.SPEC_C128
    rng = np.random.default_rng(n + 10 * Dx + 1000 * Dy)
    Sx, Sy = 2 * Dx + 1, 2 * Dy + 1
    Z = rng.standard_normal((Sy, Sx, n, n)) + 1j * rng.standard_normal((Sy, Sx, n, n))
    Gx, Gy = (max(2, 1 << (S - 1).bit_length()) for S in (Sx, Sy))
    tdt = torch.complex64 if c64 else torch.complex128
    # a guard of one more grid behind the spectra
    out = torch.full((n * n + 1, Gy, Gx), 3.0, dtype=tdt, device="cuda:0")
    r3m.r3m_build_spectral(ctx, torch.from_numpy(Z).to("cuda:0"), n, Dx, Dy, sd, out)
    E = np.zeros((Gy, Gx, n, n), complex)
    E[np.ix_(np.arange(-Dy, Dy + 1) % Gy, np.arange(-Dx, Dx + 1) % Gx)] = Z
    ref = np.fft.fft2(E, axes=(0, 1)).transpose(2, 3, 0, 1).reshape(n * n, Gy, Gx)
    got = out.cpu().numpy()
    # log2(Gx Gy) butterflies, each adding a few units of rounding to values
    # of the size of the root mean square: 1e-6 (float) and 3e-15 (double) of
    # the largest
    assert np.abs(got[:-1] - ref).max() <= (1e-6 if c64 else 3e-15) * np.abs(ref).max()
    assert np.all(got[-1] == 3.0)
    ctx.close()


def test_odd_unit_costs_what_its_neighbour_does():
    """83 bases (an odd count of shared ones) against 80: 1.08 times the work."""
    from paper_2112_05082_amd import pipeline, r3m
    ctx, D, t = r3m.Context(0), 31, {}
    for n in (80, 83):
        Z = torch.randn((2 * D + 1) ** 2, n, n, dtype=torch.complex128, device="cuda:0")
        spec = pipeline.empty_bytes(r3m.spectral_bytes(n, D, D, r3m.SPEC_C64), "cuda:0")
        times = []
        for _ in range(7):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                r3m.r3m_build_spectral(ctx, Z, n, D, D, r3m.SPEC_C64, spec)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        t[n] = min(times)
    assert t[83] < 3 * t[80], t
    ctx.close()
