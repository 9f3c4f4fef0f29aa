"""float32 layers of more than 32 channels whose sums are long are multiplied in float16 halves: sampled positions against 64
bits, at the shortest rows and ranges that take that path, with values of every scale, scales that change along a sum,
pixels far darker than their neighbours, values and weights that the halves cannot carry."""
import numpy as np
import pytest

import paper_1704_04313_amd as cb
from paper_1704_04313_amd import binding
from workloads.networks import conv, make_weights

from gpu_util import to_dev
from test_gpu_tile_shapes import _sampled

pytestmark = pytest.mark.gpu


def _scaled(x, kind):
    C, H, W = x.shape
    if kind == "large":
        return x * np.float32(2.0 ** 60)
    if kind == "small":
        return x * np.float32(2.0 ** -70)
    if kind == "brighter":  # along every sum that crosses the middle, by eight binades, and from nothing at all at the top
        x[:, : H // 2] *= np.float32(2.0 ** -8)
        x[:, : H // 5] = 0
    if kind == "dim":
        x[:, H // 4: H // 2, W // 4: W // 2] *= np.float32(2.0 ** -20)
    if kind == "special":
        for n, v in enumerate((np.nan, np.inf, -np.inf, 3.4028e38, 1e25, -1e8)):
            x[(7 * n) % C, (n * H) // 7, (n * W) // 6] = v
    return x


# 24 slices are the fewest of a whole tile, 27 and 37 leave halves of a chunk; 213 to 269 tiles are cut across, below or
# above a round of 256; 64->256 in three ranges; 100, 130 and 200 channels pad their tiles; the last three are the 64-channel
# kernels of either tile in parts
@pytest.mark.parametrize("cin,cout,k,h,w", [
    (256, 128, 3, 190, 181), (96, 100, 3, 181, 190), (84, 130, 3, 131, 129), (24, 200, 7, 133, 127), (64, 256, 7, 60, 80), (768, 128, 1, 181, 190),
    (16, 64, 7, 260, 257), (23, 50, 7, 365, 357), (96, 64, 3, 727, 725)])
@pytest.mark.parametrize("kind", ["plain", "large", "small", "brighter", "dim", "special"])
def test_against_64_bits(cin, cout, k, h, w, kind):
    L = conv(cin, cout, k, relu=False)
    (wt, b), = make_weights([L], cin + cout)
    b = b * 0
    if kind == "small":
        wt = wt * np.float32(2.0 ** -50)
    r = np.random.default_rng(cin + k)
    x = _scaled(np.maximum(r.standard_normal((cin, h, w), dtype=np.float32), 0), kind)
    rows = [slice(0, h // 4 - k), slice(h // 4 + k, h // 2 - k), slice(h // 2 - k, h // 2 + k), slice(h // 2 + k, h)]
    with np.errstate(all="ignore"):
        net = cb.CBInfer([L], [(wt, b)], x.shape, 0.02)
        net.set_mode(True)
        got = net.process_frame(to_dev(x)).cpu().numpy()[0].astype(np.float64)
        net.destroy()
        slices = (cin * k * k + 31) // 32
        for ys in rows:
            for xs in (slice(0, w), slice(w // 4 + k, w // 2 - k)):  # all, and where "dim" is
                yy, xx = np.mgrid[ys, xs]
                pos = (yy * w + xx).ravel()
                pos = r.choice(pos, min(250, pos.size), replace=False)
                want = _sampled(L, wt, b, x, pos)[0].astype(np.float32).astype(np.float64)
                size = _sampled(L, wt, b, np.where(np.isfinite(x), x, 0), pos)[1]
                g = got.reshape(cout, -1)[:, pos]
                np.testing.assert_array_equal(np.isnan(g), np.isnan(want))
                np.testing.assert_array_equal(np.isinf(g) * np.sign(g), np.isinf(want) * np.sign(want))
                fine = np.isfinite(want)
                err = np.abs(np.where(fine, g, 0) - np.where(fine, want, 0))
                # Formed again with the float32 instruction: a product and an addition per value, half a unit of 2^-23 each.
                # In halves: 2^-22 for each value's last bit and for what the second halves multiply to, and half a unit per
                # slice, doubled for what the matrix unit cuts off.
                per = cin * k * k + 40 if kind in ("dim", "special") else slices + 8
                assert np.all(err <= per * (2.0 ** -23 * np.where(fine, size, 0) + 2.0 ** -149))
                if kind in ("plain", "large", "small"):  # roundings of either sign add up like their square root
                    assert np.linalg.norm(err) <= np.sqrt(slices + 8) * 2.0 ** -24 * np.linalg.norm(want)


@pytest.mark.parametrize("kind", ["some", "channels", "inf", "zero"])
def test_weights_that_halves_do_not_carry(kind):
    """Weights far below the layer's largest where nothing else meets the pixels, infinite ones, a layer of zeros."""
    L = conv(128, 128, 3, relu=False)
    (wt, b), = make_weights([L], 9)
    b = b * 0
    r = np.random.default_rng(5)
    x = r.random((128, 131, 140), dtype=np.float32)
    if kind == "some":
        wt[:64, :64] *= np.float32(2.0 ** -40)
        x[64:, :, :70] = 0
    if kind == "channels":
        wt[5] *= np.float32(2.0 ** -60)
    if kind == "inf":
        wt[7, 100, 1, 1] = np.inf
    if kind == "zero":
        wt[:] = 0
    pos = np.concatenate([np.arange(60), r.integers(0, 131 * 140, 600)])
    want, size = _sampled(L, wt, b, x, pos)
    net = cb.CBInfer([L], [(wt, b)], x.shape, 0.02)
    net.set_mode(True)
    g = net.process_frame(to_dev(x)).cpu().numpy()[0].reshape(128, -1)[:, pos].astype(np.float64)
    net.destroy()
    fine = np.isfinite(want)
    np.testing.assert_array_equal(g[~fine], want[~fine])
    assert np.all(np.abs(np.where(fine, g, 0) - np.where(fine, want, 0)) <= (128 * 9 + 8) * 2.0 ** -23 * np.where(fine, size, 0))


class _LessMemory:
    """The library with workspaces a little smaller than what a network with filters in halves takes: it runs without them."""

    def __init__(self, lib):
        self._lib = lib

    def __getattr__(self, name):
        return getattr(self._lib, name)

    def cbinfer_workspace_bytes(self, net):
        return self._lib.cbinfer_workspace_bytes(net) - 256


@pytest.fixture
def run(monkeypatch):
    """The layer's dense output, with or without filters in halves."""
    def layer(L, wt, x, halves=True):
        with monkeypatch.context() as m:
            if not halves:
                lib = _LessMemory(cb.load_library())
                m.setattr(binding, "load_library", lambda: lib)
            net = cb.CBInfer([L], [(wt, np.zeros(L.cout, np.float32))], x.shape, 0.02)
        net.set_mode(True)
        got = net.process_frame(to_dev(x)).cpu().numpy()[0].reshape(L.cout, -1).astype(np.float64)
        net.destroy()
        return got
    return layer


def _compare(run, L, wt, x, rows, columns=1):
    """Errors of sampled positions per group of output channels (and of every `columns`-th column of the map), in halves and in
    parts: neither may depend on the scale of what a group does not see."""
    slices = (L.cin * L.kh * L.kw + 31) // 32
    r = np.random.default_rng(1)
    n = x.shape[1] * x.shape[2]
    pos = np.unique(np.concatenate([np.arange(100), n - 1 - np.arange(100), r.integers(0, n, 500)]))
    want, size = _sampled(L, wt, np.zeros(L.cout, np.float32), x, pos)
    both = [run(L, wt, x, halves)[:, pos] for halves in (True, False)]
    for g in both:
        # a product and an addition per value at most (sums formed again), half a unit of 2^-23 each
        assert np.all(np.abs(g - want) <= (L.cin * L.kh * L.kw + 40) * 2.0 ** -23 * size)
    for s in rows:
        for c in range(columns):
            at = pos % x.shape[2] % columns == c
            errors = [np.linalg.norm((g[s] - want[s])[:, at]) / np.linalg.norm(want[s][:, at]) for g in both]
            # what the parts are held to (test_gpu_float32_parts.py), and the halves like them
            assert max(errors) <= np.sqrt(slices + 8) * 2.0 ** -24, errors
            # Halves: 7.0e-8 for what they leave off, 4.7e-8 for each of four slices relative to their sum (measured for single
            # instructions), 2^-25 for each time that four are added up, 50 times at most here and half as large in the mean: as
            # squares 1.6e-7.
            assert errors[0] <= 2.0 ** -22.5, errors
    return errors


_MAP = (181, 190)  # 269 tiles of 128 positions on 256 workgroups


@pytest.mark.parametrize("bright", [0, 40, 127])
@pytest.mark.parametrize("b", [8, 14, 17, 20, 26, 30, 40, 60])
@pytest.mark.parametrize("weights", ["zero", "smaller", "positive"])
def test_one_channel_brighter(run, bright, b, weights):
    """A channel whose values are 2^b times the others', with weights that are zero or smaller by as much; or zero beside weights
    that are all positive, whose sums are large beside what each of their values is off by."""
    L = conv(128, 128, 3, relu=False)
    (wt, _), = make_weights([L], 21)
    x = np.maximum(np.random.default_rng(b).standard_normal((128,) + _MAP, dtype=np.float32), 0)
    x[bright] *= np.float32(2.0 ** b)
    wt[:, bright] *= np.float32(2.0 ** -b if weights == "smaller" else 0)
    if weights == "positive":
        wt = np.abs(wt)
    _compare(run, L, wt, x, [slice(None)])


@pytest.mark.parametrize("cin,cout,k,h,w", [(256, 128, 3) + _MAP, (64, 64, 5, 260, 257)])
@pytest.mark.parametrize("k2", [-40, -30, -24, -20, -16, -12, 16, 24, 40])
def test_two_groups(run, cin, cout, k, h, w, k2):
    """Filters of two groups, each of which sees half of the channels: the second half's values are 2^k2 of the first one's."""
    L = conv(cin, cout, k, relu=False)
    (wt, _), = make_weights([L], 22)
    x = np.maximum(np.random.default_rng(5).standard_normal((cin, h, w), dtype=np.float32), 0)
    x[cin // 2:] *= np.float32(2.0 ** k2)
    wt[: cout // 2, cin // 2:] = 0
    wt[cout // 2:, : cin // 2] = 0
    _compare(run, L, wt, x, [slice(0, cout // 2), slice(cout // 2, cout)])


@pytest.mark.parametrize("k2", [-16, -20, -30, -40])
def test_one_column_of_taps(run, k2):
    """Filters of one column of taps on a map of bright, dim and dark columns: every sum is of one kind only, whatever lies under the
    other taps; from dark to bright it is two steps, none of which is large."""
    L = conv(192, 128, 5, relu=False)
    (wt, _), = make_weights([L], 23)
    keep = np.zeros((5, 5), np.float32)
    keep[:, 2] = 1
    x = np.maximum(np.random.default_rng(6).standard_normal((192,) + _MAP, dtype=np.float32), 0)
    x[:, :, 1::3] *= np.float32(2.0 ** (k2 // 2))
    x[:, :, 0::3] *= np.float32(2.0 ** k2)
    _compare(run, L, wt * keep, x, [slice(None)], columns=3)


def test_halves_are_used(run):
    """Different bits with and without room for the halves; a layer whose length keeps the parts takes no room for them, one
    with weights that are not finite or mostly zero leaves it alone."""
    L = conv(128, 128, 3, relu=False)
    (wt, _), = make_weights([L], 24)
    x = np.random.default_rng(7).random((128,) + _MAP, dtype=np.float32)
    assert not np.array_equal(run(L, wt, x), run(L, wt, x, False))
    for w in (np.inf, -np.inf, np.nan):
        odd = wt.copy()
        odd[5, 100, 1, 1] = w
        np.testing.assert_array_equal(run(L, odd, x), run(L, odd, x, False))
    few = wt.copy()
    few[7, 80:] = 0  # 720 weights of one row
    np.testing.assert_array_equal(run(L, few, x), run(L, few, x, False))
    few[7, 80:86] = wt[7, 80:86]  # 774
    assert not np.array_equal(run(L, few, x[:, :128, :128].repeat(2, 2)), run(L, few, x[:, :128, :128].repeat(2, 2), False))
    short = conv(48, 128, 3, relu=False)
    (ws, _), = make_weights([short], 25)
    with pytest.raises(cb.CBInferError, match="needed"):
        run(short, ws, x[:48], False)


@pytest.mark.parametrize("cin,cout,k,h,w", [(768, 128, 1, 128, 256), (768, 64, 1, 128, 256), (16, 64, 7, 256, 256)])
def test_shortest_ranges(run, cin, cout, k, h, w):
    """Where halves begin, 24 slices in whole tiles, they are as exact as the parts (within the spread from one set of weights to
    another, 5 % each way)."""
    L = conv(cin, cout, k, relu=False)
    (wt, _), = make_weights([L], 28)
    x = np.maximum(np.random.default_rng(10).standard_normal((cin, h, w), dtype=np.float32), 0)
    halves, parts = _compare(run, L, wt, x, [slice(None)])
    assert halves <= 1.05 * parts
    shorter = conv(cin * 23 // 24, cout, k, relu=False)
    with pytest.raises(cb.CBInferError, match="needed"):  # no room that it could do without
        run(shorter, wt[:, : cin * 23 // 24], x[: cin * 23 // 24], False)


@pytest.mark.parametrize("streams", [1, 2])
def test_lists_in_front_of_another_layer(streams):
    """Frames of changes in two layers whose sums are long, each of which flags the next one's: with a threshold of zero they
    are those of dense frames, up to roundings."""
    layers = [conv(64, 128, 5), conv(128, 64, 3), conv(64, 8, 1, relu=False)]
    params = make_weights(layers, 33)
    r = np.random.default_rng(streams)
    frames = [np.maximum(r.standard_normal((streams, 64) + _MAP, dtype=np.float32), 0)]
    most = frames[0].copy()
    most[:, :, : 170] += r.random(most[:, :, : 170].shape, dtype=np.float32)
    few = most.copy()
    few[-1, :, 90:94, 60:80] *= np.float32(2.0 ** -20)
    frames += [most, few, frames[0]]
    lists, dense = [cb.CBInfer(layers, params, (64,) + _MAP, 0.0, n_streams=streams) for _ in range(2)]
    dense.set_mode(True)
    for t, f in enumerate(frames):
        lists.process_frame(to_dev(f))
        dense.process_frame(to_dev(f))
        for l in range(3):
            got, want = [net.read_map(l, cb.MAP_OUTPUT).astype(np.float64) for net in (lists, dense)]
            # each side within what the parts are held to, layer by layer (50, 36 and 4 slices)
            bound = 2 * sum(np.sqrt(s + 8) for s in (50, 36, 4)[: l + 1]) * 2.0 ** -24
            assert np.linalg.norm(got - want) <= bound * np.linalg.norm(want), (t, l)
            # no position is left as it was: 2^-20 of a value that is typical
            assert np.abs(got - want).max() <= 2.0 ** -18 * np.sqrt((want ** 2).mean()), (t, l)
        if t == 2:
            assert 0 < lists.layer_counts(1)[1] < 1000
    lists.destroy()
    dense.destroy()


@pytest.mark.parametrize("b", [-10, -12, -14, -16, -18, -20, -22, -24, -30])
def test_rows_of_small_weights(run, b):
    """Some output channels whose weights are all 2^b of the layer's largest."""
    L = conv(128, 128, 3, relu=False)
    (wt, _), = make_weights([L], 26)
    wt[64:] *= np.float32(2.0 ** b)
    x = np.maximum(np.random.default_rng(8).standard_normal((128,) + _MAP, dtype=np.float32), 0)
    _compare(run, L, wt, x, [slice(0, 64), slice(64, 128)])


@pytest.mark.parametrize("kind", ["outlier", "one of eight", "one of eight in small rows", "one per row"])
@pytest.mark.parametrize("b", [-10, -14, -16, -20, -24, -40])
def test_small_weights_beside_large_ones(run, kind, b):
    """One weight beside which all others are small; seven of eight consecutive channels with small weights, whose large one meets
    zeros; the same in rows that are small themselves, and with one large weight per row."""
    L = conv(128, 128, 3, relu=False)
    (wt, _), = make_weights([L], 27)
    x = np.maximum(np.random.default_rng(9).standard_normal((128,) + _MAP, dtype=np.float32), 0)
    if kind == "outlier":
        wt[3, 3, 1, 1] = np.float32(2.0 ** -b)
    elif kind != "one per row":
        small = np.arange(128) % 8 != 3
        wt[:, small] *= np.float32(2.0 ** b)
        wt[:, ~small] = np.copysign(np.float32(0.05), wt[:, ~small])
        if kind == "one of eight in small rows":
            wt[4:] *= np.float32(2.0 ** -16)
        x[~small] = 0
    else:
        wt *= np.float32(2.0 ** b)
        wt[:, 3, 1, 1] = 1
        x[3] = 0
    _compare(run, L, wt, x, [slice(0, 3), slice(4, 128)])
