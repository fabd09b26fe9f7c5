"""The staged line transforms behind the spectra (csrc/fft.h) at the extents
where a stage can go wrong: every in-register radix, primes and products of
primes (direct sums), extents 1, 2 and 1024, an odd number of rows (the last
has no partner), one to three axes, several fields."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _radix_sum(n):
    """Sum of the prime factors of n: no fewer terms than a line's stages add."""
    s, f = 0, 2
    while n > 1:
        while n % f == 0:
            s, n = s + f, n // f
        f += 1
    return s


@pytest.mark.parametrize("shape", [
    (2, 1, 1, 1), (2, 1, 1, 7), (1, 1, 1, 1021), (3, 1, 5, 64), (2, 1, 4, 2), (1, 3, 2, 9),
    (2, 8, 49, 96), (1, 1, 1024, 3), (2, 1, 7, 1024), (2, 2, 77, 101), (3, 16, 15, 25),
    (1, 512, 1, 5), (1, 1, 721, 60), (20, 6, 130, 34)])
def test_field_spectrum_every_radix(shape):
    from paper_1012_3632_amd import field_spectrum
    rng = np.random.default_rng(3)
    x = rng.standard_normal(shape)
    start = rng.standard_normal(shape)
    spec = torch.as_tensor(start, device="cuda").clone()
    field_spectrum(torch.as_tensor(x, device="cuda"), spec)
    ref = np.abs(np.fft.fftn(x, axes=(1, 2, 3))) ** 2
    # a stage of radix r adds r terms, so each line transform errs by at most
    # about eps sum(r) rms(X) with 6 rms as the largest entry; |X|^2 doubles it
    terms = 2 + sum(_radix_sum(n) for n in shape[1:])
    tol = 12 * np.finfo(float).eps * terms * ref.max()
    assert np.abs(spec.cpu().numpy() - start - ref).max() <= tol


@pytest.mark.parametrize("shape", [(1, 1024, 1024, 2), (2, 700, 999, 1), (3, 1023, 513, 1)])
def test_field_spectrum_of_many_rows(shape):
    """More rows per field than 2^17: the row index of a line is a division of
    numbers past 2^16."""
    test_field_spectrum_every_radix(shape)


# rows and columns that do not divide a block's share, every radix, primes, and
# a power of two along one axis only (the columns' in-place passes)
NOISE = [(17, 40, {}), (96, 101, {}), (60, 1024, {}), (1024, 77, {}), (7, 512, {}), (300, 210, {}),
         # e noise 300 times weaker than eps
         (64, 48, dict(cs2_0=1.0 / 3.0, kappa=0.0, rate_bulk=1.99999, rate_ghost=1.0)),
         (45, 64, dict(cs2_0=1.0 / 3.0, kappa=0.0, rate_bulk=1.99999, rate_ghost=1.0))]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,kw", NOISE)
def test_modeq_noise_every_split(nx, ny, kw, prec):
    from helpers import F32_TOL, F64_TOL, rel_err
    from oracle import modeq as OM
    from paper_1012_3632_amd.modeq import ModEq, ModEqParams
    d = dict(dict(rho0=1.0, kT=1e-5, cs2_0=0.265 ** 2, kappa=0.08, rate_bulk=1.2, rate_shear=1.6,
                  rate_ghost=0.9, seed=21, nx=nx, ny=ny), **kw)
    xi = ModEq(ModEqParams(precision=prec, **d)).noise(3).cpu().numpy()
    ref = OM.noise(3, OM.ModEqParams(**d))
    for got, want in ((xi[0], ref[0]), (xi[1], ref[5])):   # each against its own size
        assert rel_err(got, want) < (F64_TOL if prec == "fp64" else F32_TOL)


@pytest.mark.parametrize("nx,ny", [(101, 96), (256, 64), (33, 512)])
def test_modeq_batches_same_bits(nx, ny):
    """The rows and columns a block takes depend on the steps drawn together;
    the noise does not."""
    from paper_1012_3632_amd.modeq import ModEq, ModEqParams
    p = ModEqParams(nx=nx, ny=ny, precision="fp32", kT=1e-5, cs2_0=0.265 ** 2, kappa=0.08, seed=4)
    a, b = ModEq(p, batch=1), ModEq(p, batch=16)
    a.step(18)
    b.step(18)
    assert torch.equal(a.f, b.f)


@pytest.mark.parametrize("nx,ny", [(126, 931), (126, 1008), (130, 1021)])
def test_modeq_long_staged_columns(nx, ny):
    """FP64 columns with a direct sum, near the longest: a batch that would give
    a block two columns (more LDS than a compute unit has) draws the noise of
    single steps, and that noise is the oracle's."""
    from helpers import F64_TOL, rel_err
    from oracle import modeq as OM
    from paper_1012_3632_amd.modeq import ModEq, ModEqParams
    d = dict(nx=nx, ny=ny, rho0=1.0, kT=1e-5, cs2_0=0.265 ** 2, kappa=0.08, seed=4)
    p = ModEqParams(precision="fp64", **d)
    a, b = ModEq(p, batch=1), ModEq(p, batch=16)
    a.step(16)
    b.step(16)
    assert torch.equal(a.f, b.f)
    xi = a.noise(3).cpu().numpy()
    ref = OM.noise(3, OM.ModEqParams(**d))
    for got, want in ((xi[0], ref[0]), (xi[1], ref[5])):
        assert rel_err(got, want) < F64_TOL


@pytest.mark.parametrize("nx,ny", [(966, 3), (1008, 20), (1021, 8)])
def test_modeq_long_staged_rows(nx, ny):
    """FP64 rows with a direct sum whose one line takes more than 64 KB of LDS."""
    from helpers import F64_TOL, rel_err
    from oracle import modeq as OM
    from paper_1012_3632_amd.modeq import ModEq, ModEqParams
    d = dict(nx=nx, ny=ny, rho0=1.0, kT=1e-5, cs2_0=0.265 ** 2, kappa=0.08, seed=4)
    p = ModEqParams(precision="fp64", **d)
    a, b = ModEq(p, batch=1), ModEq(p, batch=16)
    xi = a.noise(3).cpu().numpy()
    ref = OM.noise(3, OM.ModEqParams(**d))
    for got, want in ((xi[0], ref[0]), (xi[1], ref[5])):
        assert rel_err(got, want) < F64_TOL
    a.step(16)
    b.step(16)
    assert torch.equal(a.f, b.f)


# relative rms errors of the FP32 (e, eps) noise of step 0 .. against the oracle's, when each
# field was transformed by itself over the full spectrum: what a packed pair may not exceed
NOISE_RMS = [((1024, 1024), 2.44e-7, 2.91e-7), ((128, 128), 2.17e-7, 2.21e-7), ((32, 1024), 2.12e-7, 2.15e-7),
             ((64, 1024), 2.22e-7, 5.59e-7), ((3, 1024), 1.68e-7, 1.72e-7), ((1024, 32), 2.22e-7, 2.25e-7),
             ((17, 64), 1.95e-7, 1.96e-7), ((9, 9), 1.61e-7, 1.67e-7), ((100, 1024), 3.31e-7, 6.02e-7)]


@pytest.mark.parametrize("n,e,eps", NOISE_RMS)
def test_modeq_noise_rms_error(n, e, eps):
    from oracle import modeq as OM
    from paper_1012_3632_amd.modeq import ModEq, ModEqParams
    d = dict(nx=n[0], ny=n[1], rho0=1.0, kT=1e-7, cs2_0=0.265 ** 2, kappa=0.08, seed=7)
    sim = ModEq(ModEqParams(precision="fp32", **d))
    err, ref = np.zeros(2), np.zeros(2)
    for k in range(max(2, min(400, 200000 // (n[0] * n[1])))):
        xi = sim.noise(k).cpu().numpy().astype(np.float64)
        want = OM.noise(k, OM.ModEqParams(**d))
        for i, j in enumerate((0, 5)):
            err[i] += ((xi[i] - want[j]) ** 2).sum()
            ref[i] += (want[j] ** 2).sum()
    got = np.sqrt(err / ref)
    assert got[0] <= e and got[1] <= eps, got


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("logn", range(11))
def test_modeq_power_of_two_lines(logn, prec):
    """The in-place rows and columns of every power of two (passes of 8, 4 and 2
    elements, and none), beside staged, thin and wide lines of the other axis."""
    from helpers import F32_TOL, F64_TOL, rel_err
    from oracle import modeq as OM
    from paper_1012_3632_amd.modeq import ModEq, ModEqParams
    n = 1 << logn
    for nx, ny in ((n, 3), (3, n), (n, 8), (100, n)):
        d = dict(nx=nx, ny=ny, rho0=1.0, kT=1e-5, cs2_0=0.265 ** 2, kappa=0.08, seed=6)
        sim = ModEq(ModEqParams(precision=prec, **d))
        xi = sim.noise(2).cpu().numpy()
        ref = OM.noise(2, OM.ModEqParams(**d))
        for got, want in ((xi[0], ref[0]), (xi[1], ref[5])):
            assert rel_err(got, want) < (F64_TOL if prec == "fp64" else F32_TOL), (nx, ny)
