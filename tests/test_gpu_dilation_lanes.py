"""Update lists of maps so large that one, two or four lanes form a word of the dilated map, of a bitmap (the frame's
changes) and of a byte map (the changes behind a layer), against the dilation that a max-pooling of the change map is."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

import paper_1704_04313_amd as cb
from workloads.networks import conv, pool

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


def positions(mask):  # [S][1][H][W] -> ascending indices
    return np.flatnonzero(mask.reshape(-1).numpy() > 0)


# rows of a few words and of many, whole words per row, less than a word per row, streams that begin inside a word
@pytest.mark.parametrize("h,w,k,stride,pooled,streams", [
    (2730, 2802, 1, 1, True, 1), (2048, 4096, 1, 1, True, 1), (2049, 2055, 3, 1, False, 1), (1930, 1954, 3, 1, True, 1),
    (250001, 17, 3, 1, False, 1), (128, 131, 4, 1, False, 260), (1449, 1451, 7, 1, False, 1), (1152, 1730, 7, 1, True, 1),
    (1835, 1841, 5, 2, False, 1), (33, 70, 8, 1, False, 950)])
@pytest.mark.parametrize("behind", [False, True])  # a 1x1 layer that passes the frame on
def test_lists(h, w, k, stride, pooled, streams, behind):
    pad = (k - 1) // 2
    layers = ([conv(1, 1, 1)] if behind else []) + [conv(1, 1, k, stride=stride)] + ([pool()] if pooled else [])
    params = [None if L.kind == "pool" else (np.ones((1, 1, L.kh, L.kw), np.float32), np.zeros(1, np.float32)) for L in layers]
    r = np.random.default_rng(h + k)
    a = torch.zeros((streams, 1, h, w))
    changed = torch.zeros((streams, 1, h, w))
    for _ in range(60):  # solid blocks and lone pixels, some at the edges
        s, y, x = int(r.integers(0, streams)), int(r.integers(0, h)), int(r.integers(0, w))
        changed[s, 0, y:y + int(r.integers(1, 40)), x:x + int(r.integers(1, 200))] = 1
        changed[int(r.integers(0, streams)), 0, int(r.integers(0, h)), int(r.integers(0, w))] = 1
    changed[0, 0, 0, 0] = changed[-1, 0, -1, -1] = 1
    net = cb.CBInfer(layers, params, (1, h, w), 0.5, n_streams=streams)
    try:
        net.process_frame(to_dev(a.numpy()))
        net.process_frame(to_dev(changed.numpy()))
        l = 1 if behind else 0
        update = F.max_pool2d(changed, k, stride, pad)
        np.testing.assert_array_equal(net.read_list(l, cb.LIST_CHANGED), positions(changed))
        np.testing.assert_array_equal(net.read_list(l, cb.LIST_UPDATE), positions(update))
        if pooled:
            np.testing.assert_array_equal(net.read_list(l + 1, cb.LIST_UPDATE), positions(F.max_pool2d(update, 2)))
    finally:
        net.destroy()
