"""Detection leaves pieces of the stored frame unwritten that hold the same bits already: the change lists of several frames,
which the stored values decide, for each channel count, with steps below the threshold, changes of the sign of zero, and NaN."""
import numpy as np
import pytest

import paper_1704_04313_amd as cb
from workloads.networks import conv

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c,h,w,hold", [
    (1, 515, 511, False), (2, 513, 515, True), (3, 513, 513, False), (3, 2701, 2903, False), (3, 2701, 2903, True), (5, 515, 513, False),
    (6, 513, 517, True), (7, 611, 513, False),  # whole bytes per pixel, through LDS
    (3, 61, 83, False), (4, 600, 511, False), (4, 61, 83, True)])  # 16-byte units
def test_lists_over_small_steps(c, h, w, hold):
    _compare(c, h, w, hold, cb.F32)


# pieces of 256 pixels in bfloat16: a few and many, the last one short; the steps are exact in bfloat16
@pytest.mark.parametrize("c,h,w,hold", [(1, 17, 15, False), (3, 61, 83, True), (3, 515, 513, False), (8, 300, 257, False), (8, 61, 83, True)])
def test_lists_over_small_steps_bfloat16(c, h, w, hold):
    _compare(c, h, w, hold, cb.BF16)


def _compare(c, h, w, hold, dtype):
    tau = 0.5
    net = cb.CBInfer([conv(c, 1, 1, relu=False)], [(np.ones((1, c, 1, 1), np.float32), np.zeros(1, np.float32))], (c, h, w), tau,
                     hold_reference=hold, dtype=dtype)
    r = np.random.default_rng(c + h)
    f = np.zeros((c, h * w), np.float32)
    ref = f.copy()
    try:
        net.process_frame(to_dev(f.reshape(1, c, h, w)))
        for t in range(6):
            f = f.copy()
            n = h * w // (4 if t == 3 else 1000)
            f[r.integers(0, c, n), r.integers(0, h * w, n)] += np.float32(0.375)  # crosses the threshold in steps when held
            f[0, -1 - t] -= np.float32(0.375)
            f[c - 1, r.integers(0, h * w, 40)] = -0.0
            if t == 2:
                f[0, r.integers(0, h * w, 5)] = np.nan
            net.process_frame(to_dev(f.reshape(1, c, h, w)))
            flag = (np.abs(f - ref) > tau).any(0)
            np.testing.assert_array_equal(net.read_list(0, cb.LIST_CHANGED), np.flatnonzero(flag), err_msg="frame %d" % t)
            ref = np.where(flag[None] | (not hold), f, ref)
    finally:
        net.destroy()
