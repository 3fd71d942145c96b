"""Window statistics through the constant test and err = S / R at the edges of their
groups: 16 samples a thread, 256 threads a workgroup (1024 for a few windows longer than
16,384 samples), windows whose first sample is far from the rest, and constant ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402

from test_gpu_parity import check_results, gpu_run  # noqa: E402


@pytest.mark.parametrize("n", [8, 255, 257, 4095, 4096, 4097, 16384, 16385, 32769])
@pytest.mark.parametrize("flags", [0, 16])           # 16: the separate kernels
def test_reference_and_constant_windows(n, flags):
    rng = np.random.default_rng(n)
    rows = [100.0 + 10.0 * (np.arange(n) % 3) + rng.normal(0, 1, n),
            np.full(n, 3.25),
            np.where(np.arange(n) == 0, 1e6, 1.0 + 0.001 * rng.normal(0, 1, n)),
            np.where(np.arange(n) == n - 1, 2.0, 1.0),             # one sample off
            1e7 + (np.arange(n) % 2)]                              # a small spread on a large mean
    x = np.stack(rows).astype(np.float32)
    tmax = min(n // 2, 40)
    lay = oracle.Layout(len(rows), 1, n, n, n, 1, tmax)
    _, res = gpu_run(x, lay, flags=flags)
    _, out = oracle.detect(x, lay)
    check_results(res, out, f"n={n} flags={flags}")
    assert [int(v) == 2 for v in res["verdict"]] == [False, True, False, False, False]
