"""The joint reduced system of the inertial solve where its gather can go wrong, against the
FP64 CPU oracle: more measurements in a window than are staged at a time (256), measurements
whose first keyframe has the higher index, and sizes on both sides of a block of 256 entries.
The bar is the suite's FP64 bar (1e-9 in the cost, 1e-8 in the states)."""
import numpy as np
import pytest

from oracle import lbaref
from paper_2511_02036_amd import synth
from tests.parity import assert_fp64_parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2511_02036_amd import lba  # noqa: E402


def _repeated(vi, times):
    """Every measurement `times` times with its share of the information."""
    n = len(vi["edge_i"])
    out = {k: np.concatenate([v] * times) if k not in ("T_cb", "g", "v", "bg", "ba", "edge_off") else v for k, v in vi.items()}
    assert len(out["edge_i"]) == n * times
    for k in ("info", "info_bg", "info_ba"):
        out[k] = out[k] / times
    return out


def _reversed(w, vi):
    """The keyframes in the opposite order."""
    K = len(w["fixed"])
    w, vi = dict(w), dict(vi)
    w["T_cw"], w["fixed"], w["obs_kf"] = w["T_cw"][::-1].copy(), w["fixed"][::-1].copy(), (K - 1 - w["obs_kf"]).astype(np.int32)
    vi["edge_i"], vi["edge_j"] = (K - 1 - vi["edge_i"]).astype(np.int32), (K - 1 - vi["edge_j"]).astype(np.int32)
    for k in ("v", "bg", "ba"):
        vi[k] = vi[k][::-1].copy()
    return w, vi


@pytest.mark.parametrize("kopt, times, backwards", [(1, 1, False), (2, 1, True), (5, 1, True), (5, 32, False), (5, 37, True)])
def test_joint_system_matches_oracle(kopt, times, backwards):
    w, vi = synth.vi_window(570 + kopt, K=kopt + 3, n_fixed=3, M=120, nobs=(2, 6), stereo_p=0.6)
    vi = _repeated(vi, times)
    if backwards:
        w, vi = _reversed(w, vi)
    print(f"case joint system kopt={kopt} measurements={len(vi['edge_i'])} backwards={backwards}", flush=True)
    g = lba.solve_inertial(w, vi, device="cuda:0")
    r = lbaref.solve_vi(w, vi)
    assert_fp64_parity(w, g["T"], g["X"], g["outlier"], g["stats"][0], r)
    for k in ("V", "BG", "BA"):
        assert np.all(np.abs(g[k] - r[k]) <= 1e-8 * np.maximum(1.0, np.abs(r[k]))), k
