"""float32 layers multiplied as sums of bfloat16 parts (every layer but those of short filter rows): the
rounding error against 64 bits over the tile shapes, and sums that are not finite."""
import numpy as np
import pytest

import paper_1704_04313_amd as cb
from workloads.networks import conv, make_weights

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


def _reference(L, w, b, x):
    import torch
    y = torch.nn.functional.conv2d(torch.from_numpy(x.astype(np.float64))[None], torch.from_numpy(w.astype(np.float64)),
                                   torch.from_numpy(b.astype(np.float64)), stride=L.stride, padding=L.pad)[0].numpy()
    return np.maximum(y, 0) if L.relu else y


def _dense(L, params, x):
    net = cb.CBInfer([L], params, x.shape, 0.02)
    try:
        net.set_mode(True)
        return net.process_frame(to_dev(x)).cpu().numpy()[0].astype(np.float64)
    finally:
        net.destroy()


# channels around the 16 / 32 / 64 / 128 channel tiles, positions around the 64 and 128 pixel tiles, rows of
# one slice to 98, taps that straddle slices (cin not a multiple of 32); the last but three has a round of whole
# tiles, larger maps are in test_gpu_tile_shapes.py
@pytest.mark.parametrize("cin,cout,k,h,w", [
    (64, 16, 3, 9, 7), (96, 16, 5, 33, 31), (64, 20, 5, 16, 16), (48, 32, 3, 65, 64), (16, 64, 7, 8, 8),
    (16, 64, 7, 129, 131), (256, 64, 1, 17, 15), (40, 33, 3, 41, 25), (64, 65, 3, 13, 10), (64, 256, 7, 12, 11),
    (24, 100, 3, 127, 129), (512, 128, 3, 5, 3), (128, 320, 1, 23, 29), (256, 130, 3, 61, 83)])
def test_error_against_64_bits(cin, cout, k, h, w):
    L = conv(cin, cout, k, relu=False)
    (wt, b), = make_weights([L], 7 * cin + cout)
    x = np.maximum(np.random.default_rng(cin + h).standard_normal((cin, h, w)), 0).astype(np.float32)
    got, want = _dense(L, [(wt, b)], x), _reference(L, wt, b, x)
    slices = (cin * k * k + 31) // 32
    # each slice's 32 products are added to the leading sum with one rounding (half a unit of 2^-23 of it at most,
    # doubled for what the matrix unit rounds inside), the corrections and the dropped products add 2^-22 once
    size = _reference(conv(cin, cout, k, relu=False), np.abs(wt), np.abs(b), np.abs(x))
    assert np.all(np.abs(got - want) <= (slices + 8) * 2.0 ** -23 * size)
    # roundings of either sign: they add up like their square root
    assert np.linalg.norm(got - want) <= np.sqrt(slices + 8) * 2.0 ** -24 * np.linalg.norm(want)


@pytest.mark.parametrize("cin,cout,k,h,w", [(64, 256, 7, 17, 19), (16, 64, 7, 40, 40), (64, 20, 5, 16, 16)])
@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan, 3.4028e38, -3.4e38])
def test_values_that_are_not_finite(cin, cout, k, h, w, special):
    L = conv(cin, cout, k, relu=False)
    (wt, b), = make_weights([L], cin)
    wt[::3] = np.round(wt[::3] * 64) / 64  # weights of one part, zeros among them
    wt[1::3, :, 0, 0] = 0.0
    x = np.random.default_rng(3).random((cin, h, w), dtype=np.float32)
    for n in range(3):
        x[(7 * n) % cin, (k * n + 1) % h, (k * n + 2) % w] = special
    with np.errstate(all="ignore"):
        want = _reference(L, wt, b, x).astype(np.float32).astype(np.float64)
    got = _dense(L, [(wt, b)], x)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(np.isinf(got) * np.sign(got), np.isinf(want) * np.sign(want))
    fine = np.isfinite(want)
    size = _reference(L, np.abs(wt), np.abs(b), np.where(np.isfinite(x), np.abs(x), 0))
    assert np.all(np.abs(got - want)[fine] <= ((cin * k * k + 40) * 2.0 ** -23 * size)[fine])


def test_padding_channels_stay_zero_beside_the_largest_values():
    """A finite pixel whose first part rounds to infinity, in front of six channels stored as eight: the two
    padding channels must stay zero, or the layer behind multiplies its zero weights with NaN."""
    layers = [conv(64, 6, 5, relu=False), conv(6, 8, 3, relu=False)]
    (w0, b0), (w1, b1) = make_weights(layers, 11)
    w0 = w0 * np.float32(2.0 ** -100)
    b0 = b0 * 0
    x = np.random.default_rng(2).random((64, 14, 15), dtype=np.float32)
    x[7, 4, 5] = 3.4028e38
    x[50, 13, 14] = -3.4028e38
    net = cb.CBInfer(layers, [(w0, b0), (w1, b1)], x.shape, 0.02)
    got = net.process_frame(to_dev(x)).cpu().numpy()[0].astype(np.float64)
    net.destroy()
    mid = _reference(layers[0], w0, b0, x)
    want = _reference(layers[1], w1, b1, mid.astype(np.float32))
    size = _reference(layers[1], np.abs(w1), np.abs(b1), _reference(layers[0], np.abs(w0), b0, np.abs(x)).astype(np.float32))
    assert np.all(np.abs(got - want) <= (64 * 25 + 6 * 9 + 8) * 2.0 ** -23 * size)


@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan])
def test_weights_that_are_not_finite(special):
    """An infinite weight on a tap that lies in the zero padding of some outputs: zero times infinity is not a
    number there, infinity elsewhere."""
    L = conv(64, 20, 5, relu=False)
    (wt, b), = make_weights([L], 3)
    wt[3, 5, 0, 0] = special
    wt[17, 60, 4, 2] = special
    x = np.random.default_rng(4).random((64, 17, 16), dtype=np.float32) + np.float32(0.5)
    padded = np.pad(x, ((0, 0), (2, 2), (2, 2)))
    with np.errstate(all="ignore"):
        win = np.lib.stride_tricks.sliding_window_view(padded.astype(np.float64), (5, 5), axis=(1, 2))
        want = np.stack([(win * wt[o].astype(np.float64)[:, None, None]).sum(axis=(0, 3, 4)) + b[o] for o in range(20)])
    got = _dense(L, [(wt, b)], x)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(np.isposinf(got), np.isposinf(want))
    np.testing.assert_array_equal(np.isneginf(got), np.isneginf(want))
    fine = np.isfinite(want)
    size = _reference(L, np.where(np.isfinite(wt), np.abs(wt), 0), np.abs(b), x)
    assert fine[4].all() and np.all((np.abs(got - want) <= (64 * 25 + 8) * 2.0 ** -23 * size)[fine])


@pytest.mark.parametrize("exponent", [0, -100, -108, -111, -114, -118, -122, -126])
def test_pixels_near_the_smallest_float32(exponent):
    """Below 2^-110 a value is not the sum of its bfloat16 parts; sums of such values must be as exact as
    others all the same.  A third of the map is zero, a third holds ordinary values."""
    L = conv(64, 64, 3, relu=False)
    (wt, b), = make_weights([L], 6)
    x = np.random.default_rng(8).random((64, 20, 33), dtype=np.float32)
    x[:, :, :22] *= np.float32(2.0 ** exponent)
    x[:, :, 11:22] = 0
    got, want = _dense(L, [(wt, b * 0)], x), _reference(L, wt, b * 0, x)
    # float32 sums of 576 products whose roundings have either sign: a quarter unit each relative to the sum in
    # the mean; where the sums are subnormal each addition rounds by up to half of 2^-149
    for cols in (slice(0, 10), slice(12, 21), slice(23, 33)):
        g, e = got[:, :, cols], want[:, :, cols]
        assert np.linalg.norm(g - e) <= np.sqrt(576 / 4) * 2.0 ** -24 * np.linalg.norm(e) + np.sqrt(576 * e.size) * 2.0 ** -150


@pytest.mark.parametrize("exponent,pixels", [(0, 0), (-100, 0), (-108, 0), (-112, 0), (-116, 0), (-120, 0), (-125, 0),
                                              (-112, 30), (-120, 60), (-125, 80), (-136, 100), (-126, 126)])
def test_weights_near_the_smallest_float32(exponent, pixels):
    """The same for weights: rows of nothing but such weights, and of some among ordinary ones that meet only
    zeros.  With large pixels the sums of the scaled weights overflow."""
    L = conv(64, 64, 3, relu=False)
    (wt, b), = make_weights([L], 7)
    r = np.random.default_rng(12)
    wt[:32] *= np.float32(2.0 ** exponent)
    wt[32:, :32] *= np.float32(2.0 ** exponent)
    x = r.random((64, 20, 33), dtype=np.float32) * np.float32(2.0 ** pixels)
    x[32:, :, 11:] = 0
    got, want = _dense(L, [(wt, b * 0)], x), _reference(L, wt, b * 0, x)
    for rows, cols in ((slice(0, 32), slice(None)), (slice(32, 64), slice(0, 10)), (slice(32, 64), slice(12, 33))):
        g, e = got[rows, :, cols], want[rows, :, cols]
        # as above
        assert np.linalg.norm(g - e) <= np.sqrt(576 / 4) * 2.0 ** -24 * np.linalg.norm(e) + np.sqrt(576 * e.size) * 2.0 ** -150


@pytest.mark.parametrize("h,w", [(20, 20), (90, 160)])
def test_cost_of_a_value_that_is_not_finite(h, w):
    """One NaN pixel, and a map of nothing else, in a wide layer: the sums formed again take two to five times
    as long (measured), not a hundred times; the bound leaves room for a loaded machine."""
    import torch
    L = conv(64, 256, 7, relu=False)
    net = cb.CBInfer([L], make_weights([L], 3), (64, h, w), 0.02)
    net.set_mode(True)
    us = []
    for fill in (0, 1, 2):
        x = torch.rand((1, 64, h, w), device="cuda")
        if fill:
            x.view(-1)[slice(h * w // 2, h * w // 2 + 1) if fill == 1 else slice(None)] = float("nan")
        for _ in range(3):
            net.process_frame(x)
        net.set_profiling(True)
        for _ in range(5):
            net.process_frame(x)
        ms, n = net.read_profile(0, cb.STEP_NAMES.index("gemm"))
        net.set_profiling(False)
        us.append(1e3 * ms / n)
    net.destroy()
    assert max(us[1:]) <= 12 * us[0], us


@pytest.mark.parametrize("cout,fits", [(1536, True), (2048, False)])
def test_static_workspace_with_fewer_workgroups(cout, fits):
    """A network a little too large for the static workspace at full width runs there with half the workgroups
    per launch; sums are cut along K in other places then, so results agree within rounding.  One that fits (7
    million filter values on a small map) gives the same bits as in a workspace of its own."""
    L = conv(512, cout, 3, relu=False)
    params = make_weights([L], 5)
    assert (cb.cbinfer_workspace_bytes([L], params, (512, 10, 10)) <= 64 << 20) == fits
    x = np.random.default_rng(1).random((512, 10, 10), dtype=np.float32)
    got = []
    for static in (True, False):
        net = cb.CBInfer([L], params, (512, 10, 10), 0.02, static_workspace=static)
        got.append(net.process_frame(to_dev(x)).cpu().numpy().astype(np.float64))
        net.destroy()
    if fits:
        np.testing.assert_array_equal(got[0], got[1])
    assert np.linalg.norm(got[0] - got[1]) <= 2 * np.sqrt(144 + 8) * 2.0 ** -24 * np.linalg.norm(got[1])
