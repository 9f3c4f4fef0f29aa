"""Update maps that the multiplication derives itself from a change map (bits of the first layer, bytes of the one behind
it), ranked by words that rows begin on or, where those are too many, by words that run across rows; written out for
the pooling behind.  Small integers, so that every list and every value can be compared exactly with the oracle."""
import numpy as np
import pytest

import oracle
import paper_1704_04313_amd as cb
from workloads.networks import conv, pool

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


# words per row one, two, three and 32, the last one short or full; several threads per word, one, and two or three words
# per thread; more rows than words fit (2101); filters 1 to 16 wide, taller than the map; streams
@pytest.mark.parametrize("h,w,k,pooled,streams", [
    (60, 84, 7, True, 1), (61, 83, 7, False, 1), (2, 64, 3, True, 1), (5, 130, 16, False, 1), (9, 65, 16, False, 1),
    (2101, 17, 3, False, 1), (702, 66, 5, True, 1), (2, 2002, 15, True, 1), (680, 190, 3, True, 1), (240, 320, 7, True, 1),
    (40, 64, 7, True, 13), (11, 21, 5, False, 64), (90, 20, 4, False, 25), (6, 8, 1, False, 3)])
@pytest.mark.parametrize("cout", [8, 40])  # the kernel for short filter rows, where the filter allows, and the tile kernel
def test_lists_and_values(h, w, k, pooled, streams, cout):
    layers = [conv(3, 8, k), conv(8, cout, k)] + ([pool()] if pooled else [])
    r = np.random.default_rng(h + w + k)
    # few taps, so that sums stay exact
    params = []
    for L in layers:
        if L.kind != "conv":
            params.append(None)
            continue
        wt = r.integers(-1, 2, (L.cout, L.cin, k, k)) * (r.random((L.cout, L.cin, k, k)) < 40 / (L.cin * k * k))
        params.append((wt.astype(np.float32), r.integers(-2, 3, L.cout).astype(np.float32)))
    frames = [r.integers(0, 4, (streams, 3, h, w)).astype(np.float32)]
    for t in range(3):
        f = frames[-1].copy()
        for s in range(0, streams, 1 + t):
            y, x = int(r.integers(0, h)), int(r.integers(0, w))
            f[s, :, y:y + 1 + h // 6, x:x + 1 + w // (4 + 8 * t)] = r.integers(0, 4, (3, 1, 1))
            f[s, t % 3, int(r.integers(0, h)), int(r.integers(0, w))] += 1
        f[0, 0, 0, 0] += 1
        f[-1, 0, -1, -1] += 1
        frames.append(f)
    net = cb.CBInfer(layers, params, (3, h, w), 0.5, n_streams=streams)
    orcs = [oracle.OracleCBNet(layers, params, 0.5) for _ in range(streams)]
    try:
        for t, f in enumerate(frames):
            want = np.stack([orcs[s].process_frame(f[s]) for s in range(streams)])
            np.testing.assert_array_equal(net.process_frame(to_dev(f)).cpu().numpy(), want, err_msg="frame %d" % t)
            for l, L in enumerate(layers):
                which = "U" if L.kind == "conv" else "P"
                _, ho, wo = net.layer_shape(l)
                lists = [orcs[s].trace[l][which] + s * ho * wo for s in range(streams)]
                np.testing.assert_array_equal(net.read_list(l, cb.LIST_UPDATE), np.concatenate(lists),
                                              err_msg="frame %d layer %d" % (t, l))
    finally:
        net.destroy()
