"""Layers whose maps the multiplication ranks itself derive their update maps there too, also where outputs in as many rows
as the input has would be more than it ranks: filters higher than wide, padded so that the outputs are wider than the input."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_1704_04313_amd as cb
from workloads.networks import conv

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


# ranked by words that rows begin on, and by words across rows (more than 2048 of the former)
@pytest.mark.parametrize("h,w,kh,kw,pad,streams", [(7, 18724, 7, 3, 2, 1), (8, 8191, 7, 3, 2, 2), (9, 3, 9, 3, 2, 4850)])
def test_lists_and_values(h, w, kh, kw, pad, streams):
    layers = [dataclasses.replace(conv(1, 8, kh), kw=kw, pad=pad)]
    r = np.random.default_rng(h)
    params = [(r.integers(-2, 3, (8, 1, kh, kw)).astype(np.float32), r.integers(-2, 3, 8).astype(np.float32))]
    net = cb.CBInfer(layers, params, (1, h, w), 0.5, n_streams=streams)
    ho, wo = net.layer_shape(0)[1:]
    assert streams * h * wo > 131072 >= max(streams * h * w, streams * ho * wo)
    f = r.integers(0, 4, (streams, 1, h, w)).astype(np.float32)
    orcs = [oracle.OracleCBNet(layers, params, 0.5) for _ in range(streams)]
    try:
        for t in range(3):
            if t == 2:
                net.set_profiling(True)
            if t:
                f = f.copy()
                f.ravel()[r.integers(0, f.size, 300)] += 1
                f[0, 0, 0, 0] += 1
                f[-1, 0, -1, -1] += 1
            want = np.stack([orcs[s].process_frame(f[s]) for s in range(streams)])
            np.testing.assert_array_equal(net.process_frame(to_dev(f)).cpu().numpy(), want, err_msg="frame %d" % t)
            lists = [orcs[s].trace[0]["U"] + s * ho * wo for s in range(streams)]
            np.testing.assert_array_equal(net.read_list(0, cb.LIST_UPDATE), np.concatenate(lists), err_msg="frame %d" % t)
        assert net.read_profile(0, cb.STEP_NAMES.index("dilate"))[1] == 0
    finally:
        net.destroy()
