"""FFT scores from transforms of sample blocks (batches of nine sequences or more,
rolling suffixes) against the fp64 oracle, at the edges of their tiling: 2048
samples a block, 2048 lags a tile, one to sixteen tiles a pass of the block sums
and more in several, an odd number of sequences, windows that share samples.

Scores are within 1e-6 of the exact ones (the bound the fix-up enforces) plus the
rounding of the fp32 output; selections are the oracle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from gen import planted_trace  # noqa: E402

from test_gpu_fft import check_fft_scores, fft_flag, fft_parity  # noqa: E402
from test_gpu_parity import check_results  # noqa: E402

BLOCK = 4096          # points a transform: what describe_plan reports for such plans


def plan_len(lay):
    import paper_2201_01684_amd as pkg
    desc, _ = pkg.make_desc(lay.num_windows, lay.num_channels, lay.n, lay.window_stride,
                            lay.channel_stride, lay.tmin, lay.tmax, weights=lay.weights,
                            flags=pkg.FFT_SCORES)
    return pkg.describe_plan(desc)["fft_len"]


def batch(b, n, seed=0, sigma=1.5):
    return np.stack([planted_trace(n, 37 + 61 * k, 5, seed=seed + k, sigma=sigma)
                     for k in range(b)]).astype(np.float32)


@pytest.mark.parametrize("b,n,tmin,tmax", [
    (9, 2046, 1, 3),           # 2049 points: the smallest blocked plan, a block less two samples
    (9, 2048, 2, 1024),        # one whole block
    (10, 2049, 3, 1024),       # one sample in the second block
    (9, 4096, 2, 2047),        # one lag tile less a lag
    (9, 4096, 2, 2048),        # a whole lag tile: its last lag is n = 2048
    (9, 4100, 2, 2049),        # one lag in the second tile
    (11, 8193, 2041, 4096),    # lags from the middle of the first tile; two whole tiles
    (9, 20000, 4097, 8192),    # tiles 2 and 3 only: four tiles a pass
    (9, 33000, 16000, 16385),  # nine tiles
    (9, 66000, 32000, 33000),  # seventeen tiles: two passes, the second of one tile
])
def test_edges_of_the_tiling(b, n, tmin, tmax):
    x = batch(b, n, seed=n)
    lay = oracle.Layout(b, 1, n, n, n, tmin, tmax)
    assert plan_len(lay) == BLOCK
    fft_parity(x, lay, f"blocks b={b} n={n} T=[{tmin},{tmax}]")


def test_weighted_channels_and_a_lone_sequence():
    rng = np.random.default_rng(5)
    b, c, n = 3, 3, 6001                      # nine sequences: the last has no partner
    base = batch(b, n, seed=70, sigma=0.5)
    x = np.stack([base * s + rng.normal(0, 0.3, size=(b, n)) for s in (1.0, 0.01, 30.0)],
                 axis=1).astype(np.float32)
    lay = oracle.Layout(b, c, n, c * n, n, 2, 3000,
                        weights=np.array([1.0, 250.0, 0.003], dtype=np.float32))
    assert plan_len(lay) == BLOCK
    fft_parity(x, lay, "blocks, weighted channels")


def test_overlapping_and_strided_windows():
    x = planted_trace(40000, 211, 6, seed=8, sigma=2.0)
    for stride in (997, 3):                   # no alignment; almost the same window
        lay = oracle.Layout(13, 1, 9001, stride, 9001, 2, 3000)
        assert plan_len(lay) == BLOCK
        fft_parity(x, lay, f"blocks, stride {stride}")


def test_special_windows():
    n = 8192
    rows = [np.full(n, 123.25), planted_trace(n, 64, 4, seed=1, integer=True),
            planted_trace(n, 301, 9, seed=2, sigma=0.0), np.zeros(n)]
    rows += [np.random.default_rng(k).normal(0, 1, n) for k in range(5)]
    rows.append(np.where(np.arange(n) == 4000, 1e4, 0.0))    # one spike
    x = np.stack(rows).astype(np.float32)
    lay = oracle.Layout(len(rows), 1, n, n, n, 2, 4096)
    assert plan_len(lay) == BLOCK
    g, res, _ = fft_parity(x, lay, "blocks, special windows")
    assert np.all(g[1, np.arange(64, 4097, 64) - 2] == 0)


def test_same_scores_as_the_long_transforms():
    """Eight windows keep the long transforms: the same windows, in a batch of twelve, agree."""
    n, tmax = 30000, 7000
    x = batch(12, n, seed=300)
    out = {}
    for b in (8, 12):
        lay = oracle.Layout(b, 1, n, n, n, 2, tmax)
        assert (plan_len(lay) == BLOCK) == (b == 12)
        out[b] = fft_parity(x[:b], lay, f"{b} windows")
    assert np.allclose(out[8][0], out[12][0][:8], rtol=2.0 ** -22, atol=0)
    for f in ("period", "verdict", "t_cand", "t_low", "t_up", "n_candidates"):
        assert np.array_equal(out[8][1][f], out[12][1][f][:8]), f


def test_noalloc_takes_the_long_transforms_where_blocks_do_not_fit():
    import paper_2201_01684_amd as pkg
    b, n, tmax = 36, 120000, 4000             # long transforms 45 MB, blocks 81 MB of workspace
    desc, keep = pkg.make_desc(b, 1, n, n, n, 2, tmax, flags=fft_flag())
    assert pkg.workspace_bytes(desc) > 64 << 20
    x = torch.from_numpy(batch(b, n, seed=900)).to("cuda:0")
    lags = tmax - 1
    scores = torch.empty((b, lags), dtype=torch.float32, device="cuda:0")
    results = torch.zeros((b, pkg.RESULT_DTYPE.itemsize // 4), dtype=torch.int32, device="cuda:0")
    import ctypes
    stream = torch.cuda.current_stream()
    rc = pkg.load_library().gpoeo_pd_detect_noalloc(ctypes.byref(desc), x.data_ptr(),
                                                    scores.data_ptr(), results.data_ptr(),
                                                    stream.cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    det = pkg.Detector(x, desc, keep)
    det.run()
    torch.cuda.synchronize()
    res = pkg.results_to_numpy(results)
    for f in ("period", "verdict", "t_cand", "t_low", "t_up", "n_candidates"):
        assert np.array_equal(res[f], det.results_numpy()[f]), f
    one = oracle.Layout(1, 1, n, n, n, 2, tmax)
    o, out = oracle.detect(x[3].cpu().numpy(), one)
    check_fft_scores(scores[3:4].cpu().numpy(), o, "noalloc")
    check_results(res[3:4], out, "noalloc")


def test_several_launches():
    """263 sequences of 2^20 samples: 132 pairs, whose spectra (32 MiB a pair, 4 GiB a launch)
    take two launches, the second of four pairs and with a lone last sequence.  Windows on
    both sides of the boundary against the oracle."""
    b, n, tmin, tmax = 263, 1 << 20, 2040, 2060
    rng = np.random.default_rng(77)
    base = torch.from_numpy(planted_trace(n + 4 * b, 2050, 7, seed=7, sigma=3.0)).to("cuda:0")
    x = torch.stack([base[4 * k:4 * k + n] * (1.0 + 0.01 * k) for k in range(b)])
    x += torch.from_numpy(rng.normal(0, 1, n).astype(np.float32)).to("cuda:0")
    import paper_2201_01684_amd as pkg
    desc, keep = pkg.make_desc(b, 1, n, n, n, tmin, tmax, flags=fft_flag())
    det = pkg.Detector(x, desc, keep)
    assert (4 << 30) < det.ws_bytes < (4 << 30) + (100 << 20)      # 128 pairs' spectra, not 132
    det.run()
    torch.cuda.synchronize()
    scores, res = det.scores.cpu().numpy(), det.results_numpy()
    lay = oracle.Layout(1, 1, n, n, n, tmin, tmax)
    for w in (0, 1, 254, 255, 256, 257, 260, 261, 262):
        o, out = oracle.detect(x[w].cpu().numpy(), lay)
        check_fft_scores(scores[w:w + 1], o, f"window {w}")
        check_results(res[w:w + 1], out, f"window {w}")
