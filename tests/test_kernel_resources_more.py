"""No scratch memory in the segment form's kernels, the point order, the inertial ones and the
culling counters (no GPU needed).  k_linseg is at 252 vector registers and the largest
k_chol_tile at 256: one more value held spills, with identical results."""
import os

import pytest

from tests import test_kernel_resources as base


@pytest.mark.skipif(not os.path.exists(base.HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("src", ["k_linseg.hip", "k_updseg.hip", "k_segments.hip", "k_order.hip", "k_inertial.hip",
                                 "k_cull.hip"])
def test_more_kernels_use_no_scratch(src, tmp_path):
    base.test_hot_kernels_use_no_scratch(src, tmp_path)
