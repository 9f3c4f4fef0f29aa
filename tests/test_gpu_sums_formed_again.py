"""float32 sums that the bfloat16 parts do not give, formed again in the tiles of 256 pixels: 16, 32 and 64 channels, whole maps
of them or a few, even and odd numbers of slices, frames with and without padding channels.  Sampled positions against 64 bits."""
import numpy as np
import pytest

import paper_1704_04313_amd as cb
from workloads.networks import conv, make_weights

from gpu_util import to_dev
from test_gpu_tile_shapes import _sampled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,k,h,w", [
    (96, 16, 3, 183, 181), (64, 32, 5, 181, 183), (64, 20, 5, 181, 183), (16, 64, 7, 727, 725), (12, 60, 5, 725, 727),
    (3, 64, 9, 725, 727), (1, 32, 17, 513, 515)])  # stored without padding channels
@pytest.mark.parametrize("special", [np.nan, -np.inf, 3.4028e38])
def test_against_64_bits(cin, cout, k, h, w, special):
    L = conv(cin, cout, k, relu=False)
    (wt, b), = make_weights([L], cin + cout)
    b = b * 0
    r = np.random.default_rng(k)
    x = r.random((cin, h, w), dtype=np.float32)
    x[:, : h // 3] *= np.float32(2.0 ** -114)  # sums of nothing but values below 2^-110
    spots = [(0, 0, 0), (cin - 1, h - 1, w - 1), (cin // 2, h // 6, w // 2), (0, h // 2, w // 3), (cin - 1, 2 * h // 3, w // 5)]
    for c, y, q in spots:
        x[c, y, q] = special
    near = [(y + dy) * w + q + dq for _, y, q in spots for dy in range(-k, k + 1) for dq in (-k, -k // 2, -1, 0, 1, 2, k // 2, k)
            if 0 <= y + dy < h and 0 <= q + dq < w]
    pos = np.unique(np.concatenate([near, r.integers(0, h * w, 1200), np.arange(h * w - 70, h * w)]))
    with np.errstate(all="ignore"):
        want = _sampled(L, wt, b, x, pos)[0].astype(np.float32).astype(np.float64)
        size = _sampled(L, wt, b, np.where(np.isfinite(x), x, 0), pos)[1]
    net = cb.CBInfer([L], [(wt, b)], x.shape, 0.02)
    net.set_mode(True)
    got = net.process_frame(to_dev(x)).cpu().numpy()[0].reshape(cout, -1)[:, pos].astype(np.float64)
    net.destroy()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(np.isinf(got) * np.sign(got), np.isinf(want) * np.sign(want))
    fine = np.isfinite(want)
    # a float32 product and an addition per filter value, each rounded by half a unit of the sum so far or, where that
    # is subnormal, of 2^-149
    err = np.abs(got - want)[fine]
    assert np.all(err <= ((cin * k * k + 40) * (2.0 ** -23 * size + 2.0 ** -149))[fine])
