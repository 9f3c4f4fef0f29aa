"""The tile shapes of the multiplication on maps large enough for their big tiles and for several rounds of whole
tiles with a ragged rest that is cut along K, on real-valued data against 64 bits; positions in order, from
a list and ranked from the map; frames stored with and without padding channels."""
import numpy as np
import pytest

import oracle
import paper_1704_04313_amd as cb
from workloads.networks import conv, make_weights

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


def _sampled(L, w, b, x, pos):
    """Sum and sum of magnitudes in 64 bits at output positions `pos`: [cout][len(pos)]."""
    C, H, W = x.shape
    Wo = (W + 2 * L.pad - L.kw) // L.stride + 1
    p = np.pad(x, ((0, 0), (L.pad, L.pad), (L.pad, L.pad)))
    y0, x0 = pos // Wo * L.stride, pos % Wo * L.stride
    j, i = np.meshgrid(np.arange(L.kh), np.arange(L.kw), indexing="ij")
    win = p[:, y0[:, None] + j.ravel()[None], x0[:, None] + i.ravel()[None]].astype(np.float64)  # [C][n][taps]
    win = win.transpose(1, 0, 2).reshape(pos.size, -1)
    m = w.reshape(L.cout, -1).astype(np.float64)
    return m @ win.T + b[:, None].astype(np.float64), np.abs(m) @ np.abs(win.T) + np.abs(b[:, None])


def _frames(C, H, W, seed):
    r = np.random.default_rng(seed)
    a = np.maximum(r.standard_normal((C, H, W), dtype=np.float32), 0)
    half = a.copy()  # a list of about half the positions
    half[:, :H // 2] += r.random((C, H // 2, W), dtype=np.float32) + np.float32(0.1)
    few = half.copy()
    few[:, H // 3:H // 3 + 7, 3:W // 2] += np.float32(0.5)
    return [a, half, few]


# float32 rows: the 16- and 32-channel tiles (256 pixels), 64 channels at 128 and 256 pixels, 128 channels; bfloat16 the
# same.  The maps give two or three rounds of whole tiles on 256 workgroups and a rest.
@pytest.mark.parametrize("cin,cout,k,h,w,bf16", [
    (64, 16, 3, 363, 365, False), (48, 32, 3, 363, 365, False), (64, 20, 5, 257, 259, False), (32, 64, 3, 257, 259, False),
    (16, 64, 7, 725, 727, False), (24, 100, 3, 257, 259, False), (64, 256, 7, 83, 101, False),
    (64, 16, 3, 363, 365, True), (96, 32, 3, 363, 365, True), (16, 64, 7, 363, 365, True), (32, 64, 5, 161, 163, True),
    (24, 100, 7, 257, 259, True),
    # few positions: every tile cut along K, into 24, 85 and (unevenly, across tiles) six or seven parts
    (128, 32, 7, 19, 32, False), (512, 16, 7, 20, 17, False), (96, 32, 5, 67, 41, False), (128, 32, 7, 19, 32, True),
    (512, 16, 7, 20, 17, True), (192, 32, 5, 67, 41, True),
    # frames of 2^18 positions and more in float32 are stored without padding channels: units at any word
    (3, 64, 7, 515, 513, False), (3, 64, 7, 725, 727, False), (1, 20, 9, 513, 515, False), (2, 128, 5, 515, 517, False),
    (3, 16, 11, 515, 513, False), (5, 64, 5, 513, 515, False), (7, 32, 7, 515, 513, False)])
def test_against_64_bits(cin, cout, k, h, w, bf16):
    L = conv(cin, cout, k, relu=False)
    (wt, b), = make_weights([L], cin + cout + k)
    frames = _frames(cin, h, w, cin + h)
    if bf16:
        wt, frames = oracle.round_bf16(wt.copy()), [oracle.round_bf16(f.copy()) for f in frames]
    N = h * w
    r = np.random.default_rng(7)
    pos = np.unique(np.concatenate([np.arange(130), N - 1 - np.arange(300), r.integers(0, N, 1500)]))
    want = [_sampled(L, wt, b, f, pos) for f in frames]
    slices = (cin * k * k + 31) // 32
    runs = {"dense": {}, "ranked": {}, "listed": {"lists_every_frame": True}}
    if N > 131072:
        del runs["ranked"]  # lists are used either way
    first = None
    for name, kw in runs.items():
        net = cb.CBInfer([L], [(wt, b)], (cin, h, w), 0.02, dtype=cb.BF16 if bf16 else cb.F32, **kw)
        net.set_mode(name == "dense")
        for t, f in enumerate(frames):
            got = net.process_frame(to_dev(f)).cpu().numpy()[0].reshape(cout, N)
            g = got[:, pos].astype(np.float64)
            sums, size = want[t]
            if bf16:
                # rounded once to 8 bits; the 64 products that enter the accumulator together with one rounding, as below
                assert np.all(np.abs(g - sums) <= 2.0 ** -8 * np.abs(sums) + (slices + 8) * 2.0 ** -23 * size), (name, t)
            else:
                # a rounding of half a unit per slice, doubled for what the matrix unit rounds inside; corrections and
                # dropped products 2^-22 once; roundings of either sign add up like their square root
                assert np.all(np.abs(g - sums) <= (slices + 8) * 2.0 ** -23 * size), (name, t)
                assert np.linalg.norm(g - sums) <= np.sqrt(slices + 8) * 2.0 ** -24 * np.linalg.norm(sums), (name, t)
            if t == 0:  # everything is recomputed: the same work, the same bits
                first = got if first is None else first
                np.testing.assert_array_equal(got, first)
        net.destroy()
