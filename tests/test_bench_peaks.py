"""The rate that bench.py holds a layer's multiplication against is that of the instruction it runs on."""
import pytest

import bench
from workloads.networks import conv


@pytest.mark.parametrize("layer,bf16,peak", [
    (conv(3, 16, 7), False, 157.3), (conv(64, 8, 1), False, 157.3), (conv(16, 16, 3), False, 157.3),
    (conv(3, 64, 3), False, 157.3), (conv(3, 64, 7), False, 2500 / 6), (conv(3, 64, 1), False, 157.3), (conv(16, 64, 7), False, 2500 / 6),
    (conv(256, 64, 1), False, 2500 / 6), (conv(256, 16, 1), False, 157.3), (conv(3, 16, 7), True, 2500), (conv(64, 256, 7), True, 2500)])
def test_matrix_peak(layer, bf16, peak):
    assert bench.matrix_peak(layer, bf16) == pytest.approx(peak)
