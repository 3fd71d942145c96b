"""FFT scores of sequences short enough for one workgroup: transforms of up to 2048 points
(N + Tmax), and one transform of 4096 points in place of sample blocks, in rolling
detection (whose pairs may hold such a suffix window beside a longer one) and in
detection.  Against the oracle, as tests/test_gpu_rolling.py and tests/test_gpu_fft.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from gen import planted_trace  # noqa: E402

from test_gpu_rolling import check, gpu_rolling  # noqa: E402


def batch(b, c, n, periods, seed=0):
    rows = []
    for k in range(b):
        p = periods[k % len(periods)]
        rows.append(np.stack([planted_trace(n, p, min(5, p // 2 + 1), seed=seed + 10 * k + j,
                                            sigma=1.0 + j) for j in range(c)]))
    return np.stack(rows).astype(np.float32)


@pytest.mark.parametrize("b,c,n,tmax,periods", [
    (5, 1, 29, 4, [3]),                         # transforms of 64 points
    (9, 1, 512, 128, [11, 40, 90]),             # 1024 points
    (7, 1, 1638, 410, [30, 77, 200, 300]),      # the suffix plan: 1638 + 410 = 2048 points
    (7, 1, 1639, 410, [30, 77, 200, 300]),      # 2049: one transform of 4096
    (6, 1, 2731, 1365, [40, 400, 700, 900]),    # all of its 4096 points
    (5, 1, 2732, 1365, [40, 400, 700, 900]),    # 4097: sample blocks for the longest
    (3, 3, 2048, 600, [50, 250]),               # an odd number of sequences
    (11, 1, 9000, 2000, [9, 1500, 60, 390, 391, 519, 521]),  # short beside longer windows
    (3, 5, 6000, 1400, [13, 1100, 380]),        # pairs across windows and channels
])
def test_short_suffixes(b, c, n, tmax, periods):
    x = batch(b, c, n, periods, seed=n)
    w = None if c == 1 else np.array([1.0, 0.25, 3.0, 0.5, 2.0][:c], dtype=np.float32)
    lay = oracle.Layout(b, c, n, c * n, n, 1, tmax, weights=w)
    check(gpu_rolling(x, lay, "fft"), oracle.rolling(x, lay), f"{b}x{c}x{n} T<={tmax}")


@pytest.mark.parametrize("n,tmax", [
    (2046, 3), (2048, 1024),                    # 2049 points; a block
    (2731, 1365), (2732, 1365),                 # 4096 points, 4097
    (4076, 20), (4077, 20),
])
def test_one_transform_detection(n, tmax):
    """A batch of short windows: exact ties, constant rows and an odd count among them."""
    from test_gpu_fft import fft_parity
    rows = [planted_trace(n, 37 + 50 * k, 5, seed=k, sigma=1.5) for k in range(8)]
    rows += [np.full(n, 4.0), planted_trace(n, 64, 4, seed=1, integer=True),
             np.where(np.arange(n) == 700, 1e4, 0.0)]
    x = np.stack(rows).astype(np.float32)
    lay = oracle.Layout(len(rows), 1, n, n, n, 1, tmax)
    fft_parity(x, lay, f"one transform, n={n} T<={tmax}")
