"""The one-pass culling counters at the edges of a block's run, against the CPU oracle (whole
numbers: equal).  A run holds 2048 observations and looks 256 further (from 2^20 observations on), its points fill at most
sixteen LDS tiles of 4096 counters, and 512 keyframes have LDS totals; observations that are not
grouped by ascending point, and points that reach past a run's end by more, take the general
passes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import mapref  # noqa: E402
from paper_2511_02036_amd import lmap  # noqa: E402


FILL_KF, FILL_PT = 32, 1 << 17


def _check(name, counts, n_kf, levels=8, order=None, active=False, **params):
    """counts: observations per point, after 2^20 observations (512 whole runs) of other points
    by other keyframes; the oracle takes the points given, as a window of its own."""
    rng = np.random.default_rng(len(counts) + n_kf)
    pt = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    kf = rng.integers(0, n_kf, len(pt)).astype(np.int32)
    oc = rng.integers(0, levels, len(pt)).astype(np.uint8)
    if order is not None:
        i = order(rng, len(pt))
        pt, kf, oc = pt[i], kf[i], oc[i]
    fpt = np.repeat(np.arange(FILL_PT, dtype=np.int32), 8)
    fkf = rng.integers(0, FILL_KF, len(fpt)).astype(np.int32)
    foc = rng.integers(0, levels, len(fpt)).astype(np.uint8)
    act = (rng.uniform(size=len(fpt) + len(pt)) > 0.2).astype(np.uint8) if active else None
    print(f"case culling {name} N={len(pt)} points={len(counts)}", flush=True)
    got = lmap.culling(FILL_KF + n_kf, FILL_PT + len(counts), np.concatenate([fkf, kf + FILL_KF]),
                       np.concatenate([fpt, pt + FILL_PT]), np.concatenate([foc, oc]), n_levels=levels, active=act, **params)
    w = dict(fixed=np.zeros(n_kf), X=np.zeros((len(counts), 3)), obs_kf=kf, obs_pt=pt, obs_oct=oc)
    want = mapref.culling(w, n_levels=levels, active=None if act is None else act[len(fpt):], **params)
    for k in ("counters", "kf_obs", "kf_red", "cull"):
        np.testing.assert_array_equal(got[k][FILL_PT if k == "counters" else FILL_KF:], want[k], err_msg=k)
    on = np.ones(len(fpt), bool) if act is None else act[:len(fpt)] > 0
    cnt = np.bincount(fpt[on] * np.int64(levels) + foc[on], minlength=FILL_PT * levels).reshape(FILL_PT, levels)
    np.testing.assert_array_equal(got["counters"][:FILL_PT], cnt)
    np.testing.assert_array_equal(got["kf_obs"][:FILL_KF], np.bincount(fkf[on], minlength=FILL_KF))


def _swap(rng, n):
    i = np.arange(n)
    i[[2047, 4000]] = i[[4000, 2047]]   # one descent, at a run's end
    return i


@pytest.mark.parametrize("name, counts, n_kf, kw", [
    ("one observation", [1], 1, {}),
    ("a full run", [8] * 256, 20, {}),
    ("one more", [8] * 256 + [1], 20, dict(active=True)),
    ("a point over the end", [8] * 255 + [9] + [7] * 400, 20, dict(slack=1)),
    ("256 past the end", [1] * 2047 + [257] + [5] * 300, 300, {}),
    ("257 past the end", [1] * 2047 + [258] + [5] * 300, 300, {}),
    ("a point over a whole run", [3] * 100 + [2900] + [3] * 100, 3000, {}),
    ("points without observations", [0] * 700 + [6] * 300 + [0] * 5000 + [4] * 600 + [0] * 900, 30, dict(active=True)),
    ("more of them than tiles", [5] * 10 + [0] * 9000 + [5] * 500, 30, {}),
    ("many levels", [9] * 900, 40, dict(levels=32, slack=3)),
    ("one level", [9] * 900, 40, dict(levels=1)),
    ("keyframes in LDS", [4] * 1200, 512, {}),
    ("and not", [4] * 1200, 700, {}),
    ("any order", [7] * 900, 30, dict(order=lambda r, n: r.permutation(n))),
    ("one descent", [7] * 900, 30, dict(order=_swap)),
])
def test_grouped_counters_match_oracle(name, counts, n_kf, kw):
    _check(name, counts, n_kf, **kw)
