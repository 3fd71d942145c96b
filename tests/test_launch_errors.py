"""A launch that fails is reported by its entry point, whichever launch of the call it is
(CPU: the HIP runtime's launch and error functions are replaced by a preloaded stub that
launches nothing and fails the k-th launch)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <stdlib.h>
typedef struct { unsigned x, y, z; } dim3;
static int count, fail_at, last;
void stub_reset(int k) { count = 0; fail_at = k; last = 0; }
int stub_count(void) { return count; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* s) {
  (void)f; (void)g; (void)b; (void)args; (void)lds; (void)s;
  if (++count == fail_at) last = 719;          /* hipErrorLaunchFailure */
  return last;
}
int hipGetLastError(void) { int e = last; last = 0; return e; }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* s) {
  (void)g; (void)b; (void)lds; (void)s; return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** s) {
  *g = *b = (dim3){1, 1, 1}; *lds = 0; *s = 0; return 0;
}
"""

CHILD = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
from paper_2201_01684_amd import _binding as B
stub = ctypes.CDLL(sys.argv[2])
lib = B.load_library()
X, R, W = 0x100000, 0x200000, 0x300000


def call_detect(**kw):
    base = dict(num_windows=16, num_channels=1, n=20000, window_stride=20000,
                channel_stride=20000, tmin=2, tmax=4000)
    base.update(kw)
    d, keep = B.make_desc(**base)
    need = B.workspace_bytes(d)
    return lambda: (keep, lib.gpoeo_pd_detect(ctypes.byref(d), X, R, R, W, need, None))[1]


def call_rolling(**kw):
    base = dict(num_windows=16, num_channels=1, n=20000, window_stride=20000,
                channel_stride=20000, tmin=2, tmax=4000)
    base.update(kw)
    d, keep = B.make_desc(**base)
    p = B.rolling_params()
    need = B.rolling_workspace_bytes(d, p)
    return lambda: (keep, lib.gpoeo_pd_detect_rolling(ctypes.byref(d), ctypes.byref(p), X, R, W,
                                                      need, None))[1]


def call_spectral(n):
    d, keep = B.make_desc(4, 1, n, n, n, 2, n // 4)
    p = B.spectral_params(0.5)
    need = B.spectral_workspace_bytes(d, p)
    return lambda: (keep, lib.gpoeo_pd_spectral_candidates(ctypes.byref(d), ctypes.byref(p), X, R,
                                                           W, need, None))[1]


CALLS = {
    "direct": call_detect(), "unfused": call_detect(n=4096, tmax=1000, flags=B.UNFUSED),
    "tiny": call_detect(num_windows=1, n=4096, tmax=1000),
    "sliding": call_detect(num_windows=200, window_stride=2048, n=16384, channel_stride=16384),
    "fft_blocks": call_detect(flags=B.FFT_SCORES),
    "fft_long": call_detect(num_windows=2, flags=B.FFT_SCORES),
    "fft_wrap": call_detect(num_windows=2, n=16384, channel_stride=16384, flags=B.FFT_SCORES),
    "fft_small": call_detect(n=1000, tmax=300, flags=B.FFT_SCORES),
    "mfma": call_detect(flags=B.MFMA_SCORES),
    "scores_only": call_detect(flags=B.MFMA_SCORES | B.SCORES_ONLY),
    "rolling": call_rolling(), "rolling_fft": call_rolling(flags=B.FFT_SCORES),
    "rolling_fft_small": call_rolling(n=600, tmax=100, flags=B.FFT_SCORES),
    "rolling_mfma": call_rolling(flags=B.MFMA_SCORES),
    "spectral_short": call_spectral(3000), "spectral_long": call_spectral(20000),
}
for name, call in CALLS.items():
    stub.stub_reset(0)
    rc = call()
    total = stub.stub_count()
    assert rc == B.OK and total > 0, (name, rc, total)
    for k in range(1, total + 1):
        stub.stub_reset(k)
        rc = call()
        assert rc == B.EHIP, f"{name}: launch {k} of {total} failed, the call returned {rc}"
    print(name, total)
print("done")
"""


def test_every_failed_launch_is_reported(tmp_path):
    from paper_2201_01684_amd import _binding as B
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libgpoeo_pd.so is not built (run __graft_entry__.build())")
    src, lib, child = tmp_path / "stub.c", tmp_path / "stub.so", tmp_path / "child.py"
    src.write_text(STUB)
    child.write_text(CHILD)
    subprocess.run(["gcc", "-O1", "-fPIC", "-shared", str(src), "-o", str(lib)], check=True)
    r = subprocess.run([sys.executable, str(child), ROOT, str(lib)],
                       env=dict(os.environ, LD_PRELOAD=str(lib)), capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0 and "done" in r.stdout, (r.stdout + r.stderr)[-3000:]
