"""Layers of short filter rows on maps of several tiles a wave keep their taps in registers: the same bits as on a piece of the map
that is too small for that, and sampled positions against 64 bits."""
import numpy as np
import pytest

import paper_1704_04313_amd as cb
from workloads.networks import conv, make_weights

from gpu_util import to_dev
from test_gpu_tile_shapes import _sampled

pytestmark = pytest.mark.gpu


def _dense(L, params, x, bf16):
    net = cb.CBInfer([L], params, x.shape, 0.02, dtype=cb.BF16 if bf16 else cb.F32)
    net.set_mode(True)
    y = net.process_frame(to_dev(x)).cpu().numpy()[0]
    net.destroy()
    return y


# 196 608 positions are four tiles a wave; with and without padding channels, one unit to 64 per row, ragged last tiles
@pytest.mark.parametrize("cin,cout,k,stride,h,w", [
    (3, 16, 7, 1, 513, 515), (3, 16, 7, 1, 443, 445), (4, 16, 7, 1, 443, 445), (1, 5, 3, 1, 467, 469), (5, 9, 5, 1, 515, 513), (3, 16, 7, 2, 889, 887),
    (12, 16, 3, 1, 443, 447), (250, 16, 1, 1, 445, 443)])
@pytest.mark.parametrize("bf16", [False, True])
def test_same_bits_as_on_a_piece(cin, cout, k, stride, h, w, bf16):
    L = conv(cin, cout, k, relu=False, stride=stride)
    params = make_weights([L], cin + k)
    r = np.random.default_rng(h)
    x = r.random((cin, h, w), dtype=np.float32)
    got = _dense(L, params, x, bf16)
    rows = 48  # stride 2 keeps its phase
    top = _dense(L, params, x[:, :rows], bf16)
    keep = (rows - k) // stride
    np.testing.assert_array_equal(got[:, :keep], top[:, :keep])
    first = (h - rows) // 2 * 2
    bottom = _dense(L, params, x[:, first:], bf16)
    skip = k // stride + 1
    np.testing.assert_array_equal(got[:, first // stride + skip:], bottom[:, skip:])
    if not bf16:
        n = got[0].size
        pos = np.unique(np.concatenate([np.arange(60), n - 1 - np.arange(60), r.integers(0, n, 500)]))
        want, size = _sampled(L, *params[0], x, pos)
        # a product and an addition per value, half a unit each
        assert np.all(np.abs(got.reshape(cout, -1)[:, pos] - want) <= (cin * k * k + 2) * 2.0 ** -23 * size)


# lists of 196 608 positions and more, ragged ones of them, and short lists by the same kernel; one stream and two; a layer of the
# same kernel behind the first, which takes its changes from it
@pytest.mark.parametrize("streams,h,w", [(1, 515, 513), (2, 371, 359)])
@pytest.mark.parametrize("bf16", [False, True])
def test_lists_give_the_bits_of_dense_frames(streams, h, w, bf16):
    """With a threshold of zero a frame's output does not depend on what was kept from the frames before it."""
    layers = [conv(3, 16, 7), conv(16, 16, 3, relu=False)]
    params = make_weights(layers, 31)
    r = np.random.default_rng(h)
    frames = [r.random((streams, 3, h, w), dtype=np.float32)]
    most = frames[0].copy()
    most[:, :, : h * 9 // 10] += r.random(most[:, :, : h * 9 // 10].shape, dtype=np.float32)
    few = most.copy()
    few[-1, :, h // 2: h // 2 + 3, w // 3: w // 2] += np.float32(0.25)
    frames += [most, few, frames[0]]
    dtype = cb.BF16 if bf16 else cb.F32
    lists, dense = [cb.CBInfer(layers, params, (3, h, w), 0.0, n_streams=streams, dtype=dtype) for _ in range(2)]
    dense.set_mode(True)
    for t, f in enumerate(frames):
        got, want = [net.process_frame(to_dev(f)).cpu().numpy() for net in (lists, dense)]
        np.testing.assert_array_equal(got, want, err_msg="frame %d" % t)
        if t == 1:
            assert 4 * 12 * 256 * 16 <= lists.layer_counts(0)[1] < streams * h * w
        if t == 2:
            assert 0 < lists.layer_counts(0)[1] < 4 * 12 * 256 * 16
    lists.destroy()
    dense.destroy()
