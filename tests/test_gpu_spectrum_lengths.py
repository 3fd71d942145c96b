"""Amplitude spectra of every split length, 2^13 (two rows of 4096) to 2^22 points
(every sequence of column radices; 1025 chunks of bins a window), an odd number of
sequences and windows that share samples, against the oracle.  The period of 40 + 17 lg
samples or so of each trace puts its strongest peaks near L / period, and the narrow
levels of its template harmonics up to L / 2."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gen import planted_trace  # noqa: E402

from test_gpu_spectral import check, gpu_spectral  # noqa: E402


@pytest.mark.parametrize("lg", range(12, 23))
def test_every_split(lg):
    n = (1 << lg) - (lg % 3)                       # whole and ragged lengths
    b = 3 if lg < 18 else 1                        # the last pair holds one sequence
    x = np.stack([planted_trace(n, 40 + 17 * lg + 300 * k, 6, seed=lg + k, sigma=1.0)
                  for k in range(b)])
    res = gpu_spectral(x, b, 1, n, n, n, 2, n // 2, c_peak=0.3)
    check(res, x, range(b), 1, n, n, n, 2, n // 2, c_peak=0.3, where=f"L=2^{lg}")


def test_overlapping_windows_of_two_channels():
    n, stride = 9000, 701
    x = np.stack([planted_trace(30000, 211, 6, seed=1), planted_trace(30000, 211, 4, seed=2) * 3])
    res = gpu_spectral(x, 7, 2, n, stride, 30000, 2, 4000, c_peak=0.3)
    check(res, x, range(7), 2, n, stride, 30000, 2, 4000, c_peak=0.3, where="overlapping")
