"""How the tile kernel's producers address image-matrix rows: slices inside one filter tap with a bit per tap column
(filters up to 32 wide, no higher than the map), units of several taps per slice tested in 16 bits, and neither for sides
above 16000.  Every position of small maps, borders included, against 64 bits."""
import numpy as np
import pytest

import oracle
import paper_1704_04313_amd as cb
from paper_1704_04313_amd import BF16, F32
from workloads.networks import conv, make_weights

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,k,stride,h,w,dtype", [
    # one tap per slice: windows over both borders, stride, 32 columns, several slices per tap, bfloat16
    (64, 64, 7, 1, 9, 11, F32), (32, 130, 5, 2, 17, 19, F32), (32, 20, 32, 1, 33, 34, F32), (96, 64, 3, 1, 3, 200, F32),
    (64, 100, 5, 1, 23, 9, BF16), (128, 64, 3, 2, 21, 17, BF16),
    # the same channels where that does not hold: a filter 33 wide, maps of fewer rows than the filter
    (32, 20, 33, 1, 34, 36, F32), (32, 64, 3, 1, 1, 50, F32), (64, 64, 5, 1, 2, 33, BF16),
    # several taps per slice, or a slice across taps; the longest side for 16 bits
    (16, 64, 7, 1, 9, 11, F32), (20, 64, 5, 2, 13, 12, F32), (40, 33, 3, 1, 7, 70, BF16), (16, 64, 5, 1, 3, 16000, F32),
    # longer ones, across and down
    (16, 64, 5, 1, 3, 16001, F32), (24, 64, 5, 1, 16003, 2, F32), (48, 64, 3, 1, 2, 16100, BF16)])
def test_every_position(cin, cout, k, stride, h, w, dtype):
    import torch
    L = conv(cin, cout, k, relu=False, stride=stride)
    (wt, b), = make_weights([L], cin + cout)
    x = np.random.default_rng(h + w).standard_normal((cin, h, w)).astype(np.float32)
    if dtype == BF16:
        wt, x = oracle.round_bf16(wt.copy()), oracle.round_bf16(x.copy())
    args = [torch.from_numpy(v.astype(np.float64)) for v in (x[None], wt, b)]
    want = torch.nn.functional.conv2d(*args, stride=stride, padding=L.pad)[0].numpy()
    size = torch.nn.functional.conv2d(*(v.abs() for v in args), stride=stride, padding=L.pad)[0].numpy()
    net = cb.CBInfer([L], [(wt, b)], (cin, h, w), 0.02, dtype=dtype)
    for dense in (True, False):
        net.set_mode(dense)
        got = net.process_frame(to_dev(x)).cpu().numpy()[0].astype(np.float64)
        # a rounding per slice of 32 products, of half a unit doubled for what the matrix unit rounds inside; the
        # corrections and dropped products 2^-22 once; bfloat16 outputs are rounded to 8 bits
        lim = ((cin * k * k + 31) // 32 + 8) * 2.0 ** -23 * size + (2.0 ** -8 * np.abs(want) if dtype == BF16 else 0)
        assert np.all(np.abs(got - want) <= lim)
    net.destroy()
