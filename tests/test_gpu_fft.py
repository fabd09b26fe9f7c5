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
