"""The segment form of the FP64 step at its limits, against the FP64 CPU oracle.

A chunk holds 64 observations and 32 points, a segment 10 optimisable keyframes and up to
16 chunks, a range 512 positions; poses are staged in LDS up to 64 keyframes.  Beyond these the general form runs.  The sizes below lie on both sides of each
limit.  The bar is the suite's FP64 bar (1e-9 in the cost, 1e-8 in the states)."""
import numpy as np
import pytest

from oracle import lbaref
from paper_2511_02036_amd import synth
from tests.parity import assert_fp64_parity, window_slice

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2511_02036_amd import lba  # noqa: E402


def _check(w, name):
    print(f"case segments {name} N={len(w['obs_kf'])}", flush=True)
    g = lba.solve(w, device="cuda:0")
    assert_fp64_parity(w, g["T"], g["X"], g["outlier"], g["stats"][0], lbaref.solve(w))


@pytest.mark.parametrize("K, fixed, M, nobs", [
    (3, 2, 1, (2, 3)),          # one point
    (6, 2, 40, (2, 2)),         # more than 32 points before a chunk is full
    (12, 2, 150, (10, 12)),     # up to ten optimisable keyframes per point
    (13, 2, 150, (11, 13)),     # eleven: the general form
    (24, 2, 513, (2, 6)),       # a sorted window, several ranges and segments
    (64, 36, 300, (3, 8)),      # poses staged in LDS
    (65, 36, 300, (3, 8)),      # and not
    (128, 100, 300, (3, 8)),    # the most keyframes of a window
    (12, 4, 9000, (6, 9)),      # segments of several chunks
])
def test_segment_limits_match_oracle(K, fixed, M, nobs):
    w = synth.tiny_window(500 + K + M, K=K, n_fixed=fixed, M=M, nobs=nobs, stereo_p=0.6)
    _check(w, f"K={K} fixed={fixed} M={M} nobs={nobs}")


@pytest.mark.parametrize("sizes", [(1, 600, 33, 2000), (513, 512, 64)])
def test_batch_of_uneven_windows_matches_oracle(sizes):
    ws = [synth.tiny_window(540 + i, K=8 + 6 * i, n_fixed=3, M=M, nobs=(2, 7), stereo_p=0.5) for i, M in enumerate(sizes)]
    cat = synth.concat(ws)
    print(f"case segments batch {sizes} N={len(cat['obs_kf'])}", flush=True)
    g = lba.solve(cat, device="cuda:0")
    for i, w in enumerate(ws):
        ks, ps, os_ = window_slice(cat, i)
        assert_fp64_parity(w, g["T"][ks], g["X"][ps], g["outlier"][os_], g["stats"][i], lbaref.solve(w))


def test_single_precision_measurements_match_oracle():
    w = synth.tiny_window(560, K=14, n_fixed=4, M=400, nobs=(3, 8), stereo_p=0.6)
    w["obs_z"] = np.asarray(w["obs_z"]).astype(np.float32).astype(np.float64)
    print(f"case segments z_f32 N={len(w['obs_kf'])}", flush=True)
    g = lba.solve(w, device="cuda:0", z_f32=True)
    assert_fp64_parity(w, g["T"], g["X"], g["outlier"], g["stats"][0], lbaref.solve(w))
