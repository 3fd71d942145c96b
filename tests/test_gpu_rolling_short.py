"""Rolling detection by FFT where its suffix windows are short: the suffix plan's two
limits (longest window plus Tmax of 2048 points: one workgroup's transform of that length;
windows of one block of 2048 samples: one workgroup's transform of 4096 points), and
batches whose pairs hold one-block windows beside longer ones.  Against the oracle, as
tests/test_gpu_rolling.py."""
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
    (7, 1, 1639, 410, [30, 77, 200, 300]),      # 2049: one block
    (6, 1, 2048, 1024, [40, 400, 700, 900]),    # whole blocks, lag 1024
    (5, 1, 2049, 1024, [40, 400, 700, 900]),    # one sample in the second block
    (3, 3, 2048, 600, [50, 250]),               # an odd number of sequences
    (11, 1, 9000, 2000, [9, 1500, 60, 390, 391]),   # one-block windows beside longer ones
    (3, 5, 6000, 1400, [13, 1100, 380]),        # pairs across windows and channels
])
def test_short_suffixes(b, c, n, tmax, periods):
    x = batch(b, c, n, periods, seed=n)
    w = None if c == 1 else np.array([1.0, 0.25, 3.0, 0.5, 2.0][:c], dtype=np.float32)
    lay = oracle.Layout(b, c, n, c * n, n, 1, tmax, weights=w)
    check(gpu_rolling(x, lay, "fft"), oracle.rolling(x, lay), f"{b}x{c}x{n} T<={tmax}")


@pytest.mark.parametrize("n", [2046, 2048])
def test_one_block_detection(n):
    """A batch of one-block windows of more than 2048 points: exact ties, constant rows and
    an odd count among them."""
    from test_gpu_fft import fft_parity
    rows = [planted_trace(n, 37 + 50 * k, 5, seed=k, sigma=1.5) for k in range(8)]
    rows += [np.full(n, 4.0), planted_trace(n, 64, 4, seed=1, integer=True),
             np.where(np.arange(n) == 700, 1e4, 0.0)]
    x = np.stack(rows).astype(np.float32)
    lay = oracle.Layout(len(rows), 1, n, n, n, 1, n // 2)
    fft_parity(x, lay, f"one block, n={n}")
