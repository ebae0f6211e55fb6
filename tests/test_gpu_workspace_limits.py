"""The largest batches that the solver's plan accepts.  Only the plan is formed (its sizes come
from host arrays): the device arrays of the problems are never read, so one dummy stands for
them."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2511_02036_amd import lba, synth  # noqa: E402


def _workspace(windows, kopt, points=0, per_point=0, **options):
    """Workspace bytes of a batch of equal windows of kopt optimisable keyframes."""
    dummy = torch.zeros(64, dtype=torch.float64, device="cuda:0")
    p = dummy.data_ptr()
    off = lambda n: (np.arange(windows + 1, dtype=np.int64) * n).astype(np.int32)   # noqa: E731
    kf, pt, ob = off(kopt), off(points), off(points * per_point)
    fixed, sigma2 = np.zeros(windows * kopt, dtype=np.uint8), np.asarray(synth.SIGMA2, dtype=np.float64)
    prob = lba.Problem(int(kf[-1]), int(pt[-1]), int(ob[-1]), len(sigma2), p, fixed.ctypes.data, p, p, p, p, 0, 0, p, p,
                       sigma2.ctypes.data, lba.Intrinsics(*[float(x) for x in synth.CAM]))
    batch = lba.Batch(windows, 0, kf.ctypes.data, pt.ctypes.data, ob.ctypes.data)
    ctx = lba.Context(0, **options)
    n = C.c_size_t()
    ctx._check(ctx.lib.lba_workspace_size(ctx.handle, C.byref(prob), C.byref(batch), C.byref(n)), "lba_workspace_size")
    return n.value


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("windows, kopt", [(32866, 60), (450000, 16), (263000, 21)])
def test_batches_up_to_the_limit_of_packed_systems(windows, kopt, precision):
    """At most 2^31 - 1 doubles of packed reduced systems, n (n + 1) / 2 + n each."""
    n = 6 * kopt
    limit = (2 ** 31 - 1) // (n * (n + 1) // 2 + n)
    assert windows <= limit < windows * 1.01
    print(f"case limit windows={windows} kopt={kopt} {precision}", flush=True)
    assert _workspace(windows, kopt, precision=precision) > 8 * windows * n * (n + 1) // 2
    with pytest.raises(lba.LBAError, match="batch too large"):
        _workspace(limit + 1, kopt, precision=precision)


@pytest.mark.parametrize("windows, kopt, points, per_point", [(256, 26, 10000, 7), (2560, 26, 10000, 7),
                                                              (20000, 26, 10000, 7), (20000, 26, 13000, 8),
                                                              (65000, 20, 4000, 8)])
def test_batches_up_to_the_largest_index_fit_the_card(windows, kopt, points, per_point):
    """FP64 batches of up to 2^31 - 1 observations with their inputs in 288 GB."""
    n_pt = windows * points
    n = n_pt * per_point
    b = _workspace(windows, kopt, points, per_point)
    total = b + 34 * n + 24 * n_pt
    print(f"case fit observations={n} workspace={b / 1e9:.1f} GB with inputs {total / 1e9:.1f} GB", flush=True)
    assert total < 288e9
