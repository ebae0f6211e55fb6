"""The general form of the FP64 step (tiles of points, pairs of observations listed), which a
problem takes where the segment form does not suit it: a point seen by more than ten optimisable
keyframes, a repeated observation, or a segment plan over its capacities.  Against the FP64 CPU
oracle, with the form that ran asserted: a solve's `order` class is launched twice in the segment
form (order, plan) and three times in the general one (and the observations copied in order).

The bar is the suite's FP64 bar (1e-9 in the cost, 1e-8 in the states)."""
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

DEV = torch.device("cuda:0")


def _window(seed, kopt, M, nobs, fixed=4):
    return synth.make_window(np.random.default_rng(seed), trajectory="arc", K=kopt + fixed, n_fixed=fixed, M=M, nobs=nobs,
                             stereo_p=0.6)


def _pick(w, keep):
    out = dict(w)
    for k in ("obs_kf", "obs_pt", "obs_type", "obs_oct", "is_outlier_true"):
        out[k] = np.ascontiguousarray(w[k][keep])
    out["obs_z"] = np.ascontiguousarray(w["obs_z"][:, keep])
    return out


def _repeat_one(w):
    """One observation of an optimisable keyframe twice."""
    i = int(np.flatnonzero(np.asarray(w["fixed"])[w["obs_kf"]] == 0)[len(w["obs_kf"]) // 3])
    return _pick(w, np.insert(np.arange(len(w["obs_kf"])), i, i))


def _scattered(seed, kopt, M, per=5):
    """Points seen by any `per` keyframes: few points share ten, so that the plan needs far more
    segments than observations of neighbouring keyframes do."""
    w = _window(seed, kopt, M, (kopt + 4, kopt + 4))
    r = np.random.default_rng(seed).random(len(w["obs_kf"]))
    o = np.lexsort((r, w["obs_pt"]))
    pt = w["obs_pt"][o]
    first = np.concatenate([[0], np.flatnonzero(np.diff(pt)) + 1])
    rank = np.arange(len(pt)) - np.repeat(first, np.diff(np.append(first, len(pt))))
    return _pick(w, np.sort(o[rank < per]))


def _most_seen(w):
    on = np.asarray(w["fixed"])[w["obs_kf"]] == 0
    return int(np.bincount(w["obs_pt"][on], minlength=1).max())


def _run(data, vi=None, **options):
    """A solve with kernels launched one by one, and the form it took."""
    ctx = lba.Context(0, **options)
    prob = lba.DeviceProblem(data, device=DEV)
    s = lba.Solver(ctx, prob) if vi is None else lba.InertialSolver(ctx, prob, lba.DeviceInertial(vi, device=DEV))
    ctx.profile(True)
    s.run()
    return s, {2: "segments", 3: "general"}[ctx.profile_read()["order"][0]]


def _out(s):
    return dict(T=s.T_out.cpu().numpy(), X=s.X_out.cpu().numpy(), outlier=s.outlier.cpu().numpy().astype(bool),
                stats=s.stats_dicts())


def _parity(data, g, windows):
    if len(windows) == 1:
        assert_fp64_parity(windows[0], g["T"], g["X"], g["outlier"], g["stats"][0], lbaref.solve(windows[0]))
        return
    for i, w in enumerate(windows):
        ks, ps, os_ = window_slice(data, i)
        assert_fp64_parity(w, g["T"][ks], g["X"][ps], g["outlier"][os_], g["stats"][i], lbaref.solve(w))


def _same(a, b):
    for k in ("T", "X", "outlier"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    for sa, sb in zip(a["stats"], b["stats"]):
        np.testing.assert_equal(sa, sb)


def _in_index_order(s):
    """Whether the workspace holds the linearisation order (point, first observation,
    observations, place) with the points in index order."""
    pt = s.prob.obs_pt.cpu().numpy()
    n = s.prob.X.shape[0]
    first = np.searchsorted(pt, np.arange(n + 1)).astype(np.int32)
    rec = np.stack([np.arange(n), first[:-1], np.diff(first), first[:-1]], axis=1).astype(np.int32)
    return rec.tobytes() in s.ws.cpu().numpy().tobytes()


@pytest.mark.parametrize("why, kopt", [("repeat", 10), ("repeat", 11), ("repeat", 15), ("repeat", 20), ("repeat", 21),
                                       ("long", 11), ("long", 15), ("long", 20), ("long", 21),
                                       ("plan", 20), ("plan", 21)])
def test_order_of_the_general_form(why, kopt):
    """The general form sorts windows of more than 20 optimisable keyframes, whatever turned the
    segments down; the segments sort from 11."""
    if why == "repeat":
        w = _repeat_one(_window(600 + kopt, kopt, 400, (3, 8)))
    elif why == "long":
        w = _window(600 + kopt, kopt, 400, (kopt + 4, kopt + 4))
    else:
        w = _scattered(600 + kopt, kopt, 6000)
    assert (_most_seen(w) > 10) == (why == "long")
    print(f"case general order {why} kopt={kopt} N={len(w['obs_kf'])}", flush=True)
    s, form = _run(w)
    assert form == "general"
    assert _in_index_order(s) == (kopt <= 20)


def test_order_of_the_segments():
    for kopt, index_order in ((10, True), (11, False)):
        w = _window(640, kopt, 400, (3, 8))
        print(f"case segment order kopt={kopt} N={len(w['obs_kf'])}", flush=True)
        s, form = _run(w)
        assert form == "segments"
        assert _in_index_order(s) == index_order


def _check_forms(data, windows, form, vi=None, repeats=True, **options):
    """The form, parity, and the same bits from captured step graphs (where no observation is
    repeated: the general form adds repeated ones in any order)."""
    s, ran = _run(data, vi=vi, **options)
    assert ran == form
    g = _out(s)
    if vi is None:
        _parity(data, g, windows)
    s.ctx.profile(False)
    for _ in range(2 if repeats else 0):
        _same(g, _out(s.run()))
    return s, g


@pytest.mark.parametrize("nobs, setups", [((3, 8), 2), ((12, 14), 1)])
def test_every_kernel_of_a_solve_is_in_a_class(nobs, setups):
    """The segments' copy of the points by position is timed with the set-up (its way back with the
    flags)."""
    s, form = _run(_window(645, 12, 300, nobs))
    print(f"case classes {form}", flush=True)
    assert (form == "segments") == (setups == 2)
    assert s.ctx.profile_read()["setup"][0] == setups


def test_general_batch_with_and_without_records():
    """Points of more than ten optimisable keyframes in one window turn the segments down for all;
    sorted and unsorted windows, up to 24 optimisable keyframes (one copy of the camera sums per
    wavefront and no observation repeated: the same bits with chunk records and without)."""
    ws = [_window(650 + k, k, 300 + 40 * k, (3, 12 if k == 15 else 9)) for k in (3, 10, 15, 24)]
    assert [_most_seen(w) > 10 for w in ws] == [False, False, True, False]
    cat = synth.concat(ws)
    print(f"case general batch N={len(cat['obs_kf'])}", flush=True)
    _, a = _check_forms(cat, ws, "general", pair_cache=1)
    _, b = _check_forms(cat, ws, "general", pair_cache=0)
    _same(a, b)


@pytest.mark.parametrize("kopt", [11, 20, 31, 45])
def test_general_window_with_and_without_records(kopt):
    """Points seen by up to 16 keyframes; above 30 optimisable ones several passes over the camera
    blocks and one copy of the camera sums (equal to rounding only)."""
    w = _window(660 + kopt, kopt, 900, (4, 16))
    assert _most_seen(w) > 10
    print(f"case general window kopt={kopt} N={len(w['obs_kf'])}", flush=True)
    out = []
    for cache in (1, 0):
        s, form = _run(w, pair_cache=cache)
        assert form == "general"
        out.append(_out(s))
        _parity(w, out[-1], [w])
    if kopt <= 30:
        _same(*out)


@pytest.mark.parametrize("kopt", [20, 36, 50])
def test_plan_over_its_capacities_matches_oracle(kopt):
    w = _scattered(670 + kopt, kopt, 5000)
    assert _most_seen(w) <= 10
    print(f"case general plan kopt={kopt} N={len(w['obs_kf'])}", flush=True)
    s, form = _run(w)
    assert form == "general"
    _parity(w, _out(s), [w])


@pytest.mark.parametrize("why", ["repeat", "long"])
def test_inertial_window_in_the_general_form_matches_oracle(why):
    w, vi = synth.vi_window(680, K=16, n_fixed=4, M=500, nobs=(4, 16), stereo_p=0.6)
    if why == "repeat":
        w, vi = synth.vi_window(681, K=9, n_fixed=4, M=200, nobs=(3, 6), stereo_p=0.6)
        w = _repeat_one(w)
    assert (_most_seen(w) > 10) == (why == "long")
    print(f"case general inertial {why} N={len(w['obs_kf'])}", flush=True)
    s, g = _check_forms(w, [w], "general", vi=vi, repeats=why == "long")
    r = lbaref.solve_vi(w, vi)
    assert_fp64_parity(w, g["T"], g["X"], g["outlier"], g["stats"][0], r)
    for k, t in (("V", s.v_out), ("BG", s.bg_out), ("BA", s.ba_out)):
        assert np.all(np.abs(t.cpu().numpy() - r[k]) <= 1e-8 * np.maximum(1.0, np.abs(r[k]))), k


@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 16])
def test_segments_of_several_chunks_match_oracle(chunks):
    """A segment takes another chunk (about 52 observations) per 900 chunks of a window, up to 16;
    the update's block takes as many wavefronts, up to four."""
    w = _window(690 + chunks, 10, int((chunks - 0.5) * 900 * 52 / 9), (8, 10))
    n = len(w["obs_kf"])
    assert (n // 52 + 1 + 899) // 900 == chunks
    print(f"case segments of {chunks} chunks N={n}", flush=True)
    _check_forms(w, [w], "segments")


def test_segments_are_planned_for_two_steps_or_more():
    """A solve of at most one step lists its pairs; the workspace has one size for all."""
    w = _window(646, 12, 400, (3, 8))
    sizes, launches = set(), []
    for iters in ((0, 0), (1, 0), (0, 1), (1, 1), (2, 0)):
        print(f"case steps {iters}", flush=True)
        ctx = lba.Context(0, iters_round1=iters[0], iters_round2=iters[1])
        s = lba.Solver(ctx, lba.DeviceProblem(w, device=DEV))
        sizes.add(s.ws_bytes)
        ctx.profile(True)
        g = _out(s.run())
        prof = ctx.profile_read()
        launches.append((prof["order"][0], prof["setup"][0]))
        assert_fp64_parity(w, g["T"], g["X"], g["outlier"], g["stats"][0],
                           lbaref.solve(w, iters_round1=iters[0], iters_round2=iters[1]))
    assert len(sizes) == 1
    assert launches == [(2, 1)] * 3 + [(2, 2)] * 2   # (order and copy, or order and plan with the points' copy)


def _expected_order(w):
    """Points by lowest, then highest optimisable keyframe (none last), ties by index."""
    opt = np.where(np.asarray(w["fixed"]) == 0, np.cumsum(np.asarray(w["fixed"]) == 0) - 1, -1)
    k = opt[w["obs_kf"]]
    M, none = len(w["X"]), int((opt >= 0).sum())
    lo, hi = np.full(M, none), np.full(M, -1)
    np.minimum.at(lo, w["obs_pt"][k >= 0], k[k >= 0])
    np.maximum.at(hi, w["obs_pt"][k >= 0], k[k >= 0])
    hi[lo == none] = none
    return np.lexsort((np.arange(M), hi, lo))


@pytest.mark.parametrize("windows, M", [(1, 7272), (1, 7273), (8, 7273), (9, 7273), (1, 49152), (1, 49153), (2, 1025)])
def test_both_sorts_give_the_order(windows, M):
    """A block per lowest keyframe (up to 8 windows, 160,000 points times optimisable keyframes or
    more in the largest: 7,273 points at 22), or one block per window (digits in LDS up to 49,152
    points)."""
    ws = [_window(700 + i, 22, M if i == 0 else 60 + i, (2, 4)) for i in range(windows)]
    cat = synth.concat(ws)
    print(f"case sort windows={windows} M={M}", flush=True)
    ctx = lba.Context(0, iters_round1=0, iters_round2=0, precision="mixed")
    s = lba.Solver(ctx, lba.DeviceProblem(cat, device=DEV)).run()
    rec, p0, o0 = [], 0, 0
    for w in ws:
        order = _expected_order(w)
        n = np.bincount(w["obs_pt"], minlength=len(w["X"]))
        first = np.concatenate([[0], np.cumsum(n)])[:-1]
        place = np.concatenate([[0], np.cumsum(n[order])])[:-1]
        rec.append(np.stack([p0 + order, o0 + first[order], n[order], o0 + place], axis=1))
        p0, o0 = p0 + len(w["X"]), o0 + len(w["obs_kf"])
    assert np.concatenate(rec).astype(np.int32).tobytes() in s.ws.cpu().numpy().tobytes()


def test_sort_of_a_batch_costs_little_more_than_of_a_window():
    """96 windows fill a third of the card with a block each: 1.6 times one window (1.65 with one
    block per window for any batch; 4.1 with a block per lowest keyframe for any)."""
    w = _window(720, 42, 3000, (4, 8))   # (one block per window either way: 126,000)
    us = []
    for n in (1, 96):
        print(f"case sort time windows={n}", flush=True)
        ctx = lba.Context(0, iters_round1=0, iters_round2=0, precision="mixed")
        s = lba.Solver(ctx, lba.DeviceProblem(synth.concat([w] * n), device=DEV)).run()
        t = []
        for _ in range(6):
            ctx.profile(True)
            s.run()
            t.append(ctx.profile_read()["order"][1])
        us.append(min(t))
    assert us[1] <= 2.6 * us[0], us
