"""The bytes that bench.py counts for a launch are those that the library moves: detection leaves pieces of the stored frame
unwritten that hold the same bits already, and the output's copy has a launch of its own or is part of two others."""
import types

import numpy as np
import pytest
import torch

import bench
from workloads.networks import conv


def _frames(c, h, w, streams=1):
    return torch.from_numpy(np.random.default_rng(c).random((streams, c, h, w), dtype=np.float32))


def test_write_share_counts_pieces_of_256_pixels():
    a = _frames(3, 40, 100, 2)
    assert bench.write_share(a, a, False) == 0.0
    b = a.clone()
    b[0, 1, 0, 3] += 1  # the first piece of 31 and a quarter (2 * 4000 pixels)
    assert bench.write_share(a, b, False) == pytest.approx(256 / 8000)
    b[1, 2, 39, 99] += 1  # the last piece, 64 pixels
    assert bench.write_share(a, b, False) == pytest.approx((256 + 64) / 8000)
    b[0, 0, 39, 99] += 1  # pieces run across the border between two streams
    assert bench.write_share(a, b, False) == pytest.approx((256 + 64 + 256) / 8000)
    assert bench.write_share(a, a + 1, False) == 1.0


def test_write_share_compares_bits_of_the_storage_type():
    a = torch.ones((1, 3, 16, 32))
    b = a * (1 + 2.0 ** -12)
    assert bench.write_share(a, b, False) == 1.0 and bench.write_share(a, b, True) == 0.0
    a[:] = 0.0
    assert bench.write_share(a, -a, False) == 1.0  # the sign of zero


@pytest.mark.parametrize("c,h,w,bf16,asks", [(4, 9, 9, False, True), (5, 9, 9, False, False), (5, 512, 512, False, True),
                                              (8, 512, 512, False, False), (9, 512, 512, False, False), (8, 9, 9, True, True), (9, 9, 9, True, False)])
def test_frames_of_several_units_are_always_written(c, h, w, bf16, asks):
    a = _frames(c, h, w)
    assert bench.write_share(a, a, bf16) == (0.0 if asks else 1.0)


@pytest.mark.parametrize("launch", [False, True])
def test_bytes_of_detection_and_output(launch):
    cfg = types.SimpleNamespace(layers=[conv(3, 8, 1)], n_streams=2, dtype="f32")
    net = types.SimpleNamespace(layer_shape=lambda l: (8, 10, 20))
    prof = {(0, "detect"): (1e-3, 5), (0, "gemm"): (1e-3, 5)}
    if launch:
        prof[(0, "output")] = (1e-3, 5)
    k, _ = bench.kernel_entries(cfg, net, prof, {0: np.array([250.0, 300.0])}, 5, (3, 10, 20), detect_write=0.25)
    n = 2 * 200  # positions; 60 of them recomputed per frame
    assert k["L0.detect"]["bytes"] == n * 3 * (4 + 4 + 0.25 * 4) + n / 8 + (0 if launch else n * 8 * 8)
    assert k["L0.gemm"]["bytes"] == 4 * 24 + 4 * 3 * 60 + (4 + 4 * 8) * 60 + (0 if launch else 4 * 8 * 60)
    assert ("L0.output" in k) == launch
