"""GPU parity of the rolling detection (Algorithm 3) against the oracle.

Identical: verdict, T_init, the number of suffix windows and their starts and
periods, the selected window and period, stability and the next sampling
duration.  diff to float rounding, err within 1e-4 relative.  Each case runs
with the direct scores, the FFT scores and the matrix-core scores (whose
suffix pass reads the window table in every kernel); the FFT scores of the suffix
pass take every pair of sequences by the blocks of its own suffixes, or by one transform
where they fit it, so the mixed batches below span both and, with an odd channel count,
pairs whose two sequences come from different suffix windows.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from gen import make_workload, planted_trace  # noqa: E402


MODES = ("direct", "fft", "mfma")


def gpu_rolling(x_np, lay, mode="direct", **params):
    import paper_2201_01684_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.from_numpy(np.ascontiguousarray(x_np).reshape(-1)).to("cuda:0")
    desc, keep = pkg.make_desc(lay.num_windows, lay.num_channels, lay.n, lay.window_stride,
                               lay.channel_stride, lay.tmin, lay.tmax, lay.c_lag, lay.err_max,
                               lay.weights, flags={"direct": 0, "fft": pkg.FFT_SCORES,
                                                   "mfma": pkg.MFMA_SCORES}[mode])
    det = pkg.RollingDetector(x, desc, pkg.rolling_params(**params), keep)
    det.run()
    torch.cuda.synchronize()
    return det.results_numpy()


def check(g, o, where):
    for f in ("verdict", "t_init", "n_windows", "period", "stable", "best"):
        bad = np.nonzero(g[f] != o[f])[0]
        assert bad.size == 0, f"{where}: {f} differs at {bad[:8]}: gpu {g[f][bad[:8]]} oracle {o[f][bad[:8]]}"
    assert np.all(g["smpdur_next"] == o["smpdur_next"]), where
    assert np.all(g["flags"] == 0), f"{where}: unresolved"
    for b in range(len(g)):
        k = o["n_windows"][b]
        assert np.array_equal(g["starts"][b][:k], o["starts"][b][:k]), where
        assert np.array_equal(g["periods"][b][:k], o["periods"][b][:k]), where
    assert np.allclose(g["diff"], o["diff"], rtol=1e-6, atol=0), where
    has = o["period"] > 0
    nz = has & (o["err"] != 0)
    assert np.all(g["err"][has & (o["err"] == 0)] == 0)
    assert np.all(np.abs(g["err"][nz] - o["err"][nz]) <= 1e-4 * o["err"][nz]), where


@pytest.mark.parametrize("mode", MODES)
def test_rolling_matches_oracle_on_mixed_batch(mode):
    n = 12000
    rows = [planted_trace(n, 250, 7, seed=3, sigma=4.0),              # noisy, stable
            planted_trace(n, 137, 5, seed=4, integer=True),            # exact period
            np.concatenate([planted_trace(11500, 200, 6, seed=5, sigma=1.0),
                            planted_trace(500, 290, 6, seed=6, sigma=1.0)]),   # switch
            np.full(n, 3.5),                                           # constant
            planted_trace(n, 1900, 9, seed=7, sigma=2.0)]              # few periods
    x = np.stack(rows).astype(np.float32)
    lay = oracle.Layout(len(rows), 1, n, n, n, 2, n // 2)
    g = gpu_rolling(x, lay, mode)
    o = oracle.rolling(x, lay)
    check(g, o, f"mixed {mode}")
    assert g["stable"][1] == 1 and g["period"][1] == 137
    assert o["stable"][2] == 0 and o["smpdur_next"][2] > 0     # the switch is seen


@pytest.mark.parametrize("name,kw", [
    ("w2", dict(traces=6, n=32768, tmax=8192, pmax=3000)),
    ("w3", dict(traces=4, n=32768, tmax=8192, pmax=3000)),
    ("w5", dict(traces=3, n=16384, tmax=4096, pmax=1500)),
])
@pytest.mark.parametrize("mode", MODES)
def test_rolling_reduced_workloads(name, kw, mode):
    wl = make_workload(name, **kw)
    lay = oracle.Layout.of(wl)
    g = gpu_rolling(wl.x, lay, mode)
    o = oracle.rolling(wl.x, lay)
    check(g, o, f"{name} {mode}")


def test_rolling_fft_periods_across_length_classes():
    # periods from 12 to 3000 samples in one batch: suffixes of 27 to 15,750 samples;
    # three channels, so pairs straddle suffix windows
    n = 24000
    periods = [12, 40, 100, 333, 800, 1500, 3000]
    x = np.stack([np.stack([planted_trace(n, p, 5, seed=10 * p + c, sigma=0.5 + c)
                            for c in range(3)]) for p in periods]).astype(np.float32)
    w = np.array([1.0, 0.5, 2.0], dtype=np.float32)
    lay = oracle.Layout(len(periods), 3, n, 3 * n, n, 2, n // 2, weights=w)
    o = oracle.rolling(x, lay)
    for mode in MODES:
        check(gpu_rolling(x, lay, mode), o, f"classes {mode}")
    assert list(o["t_init"]) == periods


def test_rolling_parameters_and_threshold():
    x = np.concatenate([planted_trace(11500, 200, 6, seed=5, sigma=1.0),
                        planted_trace(500, 290, 6, seed=6, sigma=1.0)]).astype(np.float32)
    lay = oracle.Layout(1, 1, x.size, x.size, x.size, 2, x.size // 2)
    for kw in (dict(diff_threshold=10.0), dict(c_measure=3.0, step=0.25, c_eval=12.0),
               dict(c_eval=0.0)):
        g = gpu_rolling(x, lay, **kw)
        o = oracle.rolling(x, lay, **kw)
        check(g, o, str(kw))
