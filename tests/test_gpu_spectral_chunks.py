"""Spectral candidates at the edges of the scan's chunks of 2048 bins: spectra of one
chunk, of one and a bin, of several; peaks on the last bin of a chunk, on the first of
the next and on both sides of it, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gen import planted_trace  # noqa: E402

from test_gpu_spectral import check, gpu_spectral  # noqa: E402


@pytest.mark.parametrize("n", [2048, 4096, 4098, 8192, 16384])     # 1, 2, 3, 3 and 5 chunks
def test_chunk_counts(n):
    x = np.stack([planted_trace(n, p, 5, seed=p, sigma=1.0) for p in (5, 31, 200)])
    res = gpu_spectral(x, 3, 1, n, n, n, 2, n // 2, c_peak=0.2)
    check(res, x, range(3), 1, n, n, n, 2, n // 2, c_peak=0.2, where=f"n={n}")


@pytest.mark.parametrize("bins", [(2047,), (2048,), (2046, 2049), (2047, 2050, 4095), (4096, 2048)])
def test_peaks_at_chunk_edges(bins):
    n = 16384
    i = np.arange(n)
    rng = np.random.default_rng(sum(bins))
    x = np.stack([100 + sum((20.0 - k) * np.cos(2 * np.pi * b * i / n + k)
                            for k, b in enumerate(bins)) + rng.normal(0, 0.5, n)
                  for _ in range(2)])
    res = gpu_spectral(x, 2, 1, n, n, n, 2, n // 2)
    check(res, x, range(2), 1, n, n, n, 2, n // 2, where=str(bins))
    assert sorted(res["bins"][0][:len(bins)]) == sorted(bins)
