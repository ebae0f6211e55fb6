"""How the culling counters take observations that are not grouped by ascending point: the same
numbers as NumPy's (whole numbers: equal), whatever the order, the edges of a run (2048
observations, and 255 or 256 of its last point past its end) and indices out of range with the
checks off; and an observation out of place at the very end costs no abandoned single pass."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2511_02036_amd import lmap  # noqa: E402

LEVELS = 8
RUN = 2048


def _data(rng, counts, n_kf):
    pt = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    return (rng.integers(0, n_kf, len(pt)).astype(np.int32), pt, rng.integers(0, LEVELS, len(pt)).astype(np.uint8))


def _reference(n_kf, n_pt, kf, pt, oc, min_obs=3, slack=0):
    """counters, kf_obs, kf_red: observations of points or octaves out of range count nowhere, of
    keyframes out of range only in the counters."""
    ok = (pt >= 0) & (pt < n_pt) & (oc < LEVELS)
    kf, pt, oc = kf[ok], pt[ok].astype(np.int64), oc[ok].astype(np.int64)
    cnt = np.bincount(pt * LEVELS + oc, minlength=n_pt * LEVELS).reshape(n_pt, LEVELS)
    others = np.cumsum(cnt, axis=1)[pt, np.minimum(oc + slack, LEVELS - 1)] - 1
    on = (kf >= 0) & (kf < n_kf)
    return cnt, np.bincount(kf[on], minlength=n_kf), np.bincount(kf[on & (others >= min_obs)], minlength=n_kf)


def _check(name, n_kf, n_pt, data):
    print(f"case culling order {name} N={len(data[0])}", flush=True)
    got = lmap.culling(n_kf, n_pt, *data, n_levels=LEVELS, check=False, min_obs=3, slack=0)
    for key, want in zip(("counters", "kf_obs", "kf_red"), _reference(n_kf, n_pt, *data)):
        np.testing.assert_array_equal(got[key].reshape(want.shape), want, err_msg=key)


@pytest.mark.parametrize("past", [1, 254, 255, 256, 257])
@pytest.mark.parametrize("where", ["middle", "end"])
def test_points_past_a_runs_end(where, past):
    runs = (1 << 20) // RUN
    counts = np.full(runs * RUN // 8, 8)
    r = runs // 2 * RUN // 8 if where == "middle" else len(counts)
    tail = np.full(300 if where == "middle" else 0, 5)
    counts = np.concatenate([counts[:r], [2], np.full(RUN - 3, 1), [1 + past], tail, counts[r:]])
    _check(f"{where} {past}", 300, len(counts), _data(np.random.default_rng(past), counts, 300))


@pytest.mark.parametrize("what", ["point", "large point", "keyframe", "octave"])
@pytest.mark.parametrize("at", [0, 2047, 2048, 700000, -1])
def test_indices_out_of_range_with_the_checks_off(what, at):
    n_pt, n_kf = (1 << 17) + 50, 900
    kf, pt, oc = _data(np.random.default_rng(3), np.full(n_pt, 8), n_kf)
    if what == "point":
        pt[at] = -5
    elif what == "large point":
        pt[at] = 0x7fffffff
    elif what == "keyframe":
        kf[at] = n_kf if at % 2 else -1
    else:
        oc[at] = 200
    _check(f"{what} {at}", n_kf, n_pt, (kf, pt, oc))


def test_a_late_descent_costs_no_abandoned_pass():
    """5 million observations: 665 us in order, 740 in general passes; 1,220 with the single pass
    abandoned at its end."""
    n_pt = 640000
    data = _data(np.random.default_rng(5), np.full(n_pt, 8), 2000)
    late = tuple(d.copy() for d in data)
    for d in late:
        d[[-1, -3000]] = d[[-3000, -1]]
    best = []
    for name, (kf, pt, oc) in (("in order", data), ("late", late)):
        print(f"case culling time {name}", flush=True)
        job = lmap.Culling(2000, n_pt, kf, pt, oc, LEVELS, device="cuda:0")
        t = []
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            job.run(check=False)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best.append(min(t))
    assert best[1] <= 1.4 * best[0], best


@pytest.mark.parametrize("n_pt, shuffled", [(3000, False), (140000, False), (140000, True)])
@pytest.mark.parametrize("first", [0, 1])
def test_protect_and_cull_in_one_array(first, n_pt, shuffled):
    """A caller's array that holds the protected keyframes and takes the culled ones."""
    n_kf = 700
    rng = np.random.default_rng(8)
    data = _data(rng, np.full(n_pt, 8), n_kf)
    if shuffled:
        i = rng.permutation(len(data[0]))
        data = tuple(d[i] for d in data)
    protect = (rng.uniform(size=n_kf) < 0.3).astype(np.uint8)
    protect[0] = first
    print(f"case culling in place first={first} N={len(data[0])} shuffled={shuffled}", flush=True)
    apart = lmap.Culling(n_kf, n_pt, *data, LEVELS, protect=protect)
    apart.run(lmap.cull_params(num=1, den=2), check=False)
    one = lmap.Culling(n_kf, n_pt, *data, LEVELS, protect=protect)
    one.cull = one.protect
    one.run(lmap.cull_params(num=1, den=2), check=False)
    a, b = apart.result(), one.result()
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    assert a["cull"][0] != first and a["cull"].any()


@pytest.mark.parametrize("n_pt", [2000, 140000])
def test_counting_is_one_launch_of_its_class_per_call(n_pt):
    """The benchmark divides a call's bytes by the class's mean: a call whose counting takes
    several kernels counts once."""
    job = lmap.Culling(300, n_pt, *_data(np.random.default_rng(2), np.full(n_pt, 8), 300), LEVELS)
    lmap.profile(True)
    for _ in range(3):
        job.run(check=False)
    prof = lmap.profile_read()
    lmap.profile(False)
    print(f"case culling profile N={8 * n_pt} {prof['cull_count']}", flush=True)
    assert [prof[k][0] for k in ("cull_count", "cull_redundant", "cull_decide")] == [3, 3, 3]
