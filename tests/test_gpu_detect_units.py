"""Change detection on frames whose pixels take several 16-byte units of the stored map: unit counts around
the waves of a workgroup and the loads a wave has in flight, pixel counts around a bitmap word."""
import numpy as np
import pytest

from workloads.networks import conv, make_weights

from gpu_util import compare_sequence

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("hold", [False, True])
@pytest.mark.parametrize("channels,h,w", [(5, 7, 9), (9, 8, 8), (16, 5, 13), (61, 16, 12), (64, 9, 7), (68, 11, 12),
                                          (130, 3, 43), (260, 10, 13), (520, 5, 5)])
def test_lists_and_stored_input(channels, h, w, hold, bf16):
    L = conv(channels, 8, 1)
    r = np.random.default_rng(channels)
    base = r.random((channels, h, w), dtype=np.float32)
    frames = [base]
    for t in range(3):
        f = frames[-1].copy()
        for p in r.integers(0, h * w, max(1, h * w // 8)):  # one channel each, above and below the threshold
            f[r.integers(0, channels), p // w, p % w] += np.float32(r.choice([0.5, -0.5, 0.01]))
        frames.append(f)
    compare_sequence([L], make_weights([L], channels), frames, 0.02, hold=hold, bf16=bf16,
                     label="%d channels on %d x %d" % (channels, w, h))
