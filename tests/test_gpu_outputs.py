"""The caller's planar output: written by the last layer itself next to a copy of what stays (small outputs), or by
a copy launch (larger ones, pooling at the end, an output in the frame's own memory).  Whatever the way, every
frame's buffer must hold the last layer's stored map, also when the buffers alternate."""
import numpy as np
import pytest

import paper_1704_04313_amd as cb
from workloads.networks import conv, make_weights, pool

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


# outputs below and above 4 MB, channels around the units and the 64 channels a copying workgroup takes, both
# multiplication kernels, ragged and single pixels, streams
@pytest.mark.parametrize("cin,cout,k,h,w,streams,pooled,dtype", [
    (3, 16, 7, 64, 64, 1, False, cb.F32), (3, 5, 3, 31, 29, 3, False, cb.F32), (40, 20, 3, 21, 19, 2, False, cb.F32),
    (64, 130, 3, 17, 23, 1, False, cb.F32), (16, 100, 5, 9, 11, 5, False, cb.BF16), (3, 6, 5, 40, 33, 2, False, cb.BF16),
    (1, 1, 1, 1, 1, 1, False, cb.F32), (3, 65, 3, 131, 127, 1, False, cb.F32), (8, 200, 3, 90, 70, 1, False, cb.BF16),
    (64, 320, 3, 61, 63, 1, False, cb.F32), (3, 24, 3, 367, 363, 1, False, cb.F32), (3, 130, 3, 64, 66, 2, True, cb.F32),
    (3, 20, 3, 64, 66, 2, True, cb.BF16)])
@pytest.mark.parametrize("dense", [False, True])
def test_output_is_the_stored_map(cin, cout, k, h, w, streams, pooled, dtype, dense):
    import torch
    layers = [conv(cin, cout, k, relu=False)] + ([pool()] if pooled else [])
    net = cb.CBInfer(layers, make_weights(layers, cout), (cin, h, w), 0.02, n_streams=streams, dtype=dtype)
    net.set_mode(dense)
    r = np.random.default_rng(cin + h)
    f = r.random((streams, cin, h, w), dtype=np.float32)
    outs = [torch.full(net.out_shape, float("nan"), device="cuda") for _ in range(2)]
    for t in range(4):
        f = f.copy()
        f[t % streams, :, t:t + 1 + h // 5, : 1 + w // 4] += np.float32(0.5)
        if t == 3:
            net.reset()
        got = net.process_frame(to_dev(f), outs[t % 2])
        np.testing.assert_array_equal(got.cpu().numpy(), net.read_map(len(layers) - 1, cb.MAP_OUTPUT), err_msg="frame %d" % t)
    net.destroy()


@pytest.mark.parametrize("shift", [0, 1, 2 * 3 * 40 * 36 - 1])
def test_output_in_the_memory_of_the_frame(shift):
    """The frame has been read when the output is written, wherever they overlap."""
    import torch
    layers = [conv(3, 8, 5), conv(8, 3, 3, relu=False)]
    params = make_weights(layers, 4)
    nets = [cb.CBInfer(layers, params, (3, 40, 36), 0.02, n_streams=2) for _ in range(2)]
    n = 2 * 3 * 40 * 36
    f = np.random.default_rng(1).random(n, dtype=np.float32)
    for t in range(3):
        f[500 * t:500 * t + 300] += np.float32(0.25)
        mem = torch.zeros(2 * n, device="cuda")
        mem[shift:shift + n] = to_dev(f)
        got = nets[0].process_frame(mem[shift:shift + n].view(2, 3, 40, 36), mem[:n].view(2, 3, 40, 36)).cpu().numpy()
        np.testing.assert_array_equal(got, nets[1].process_frame(to_dev(f).view(2, 3, 40, 36)).cpu().numpy(), err_msg="frame %d" % t)
    for net in nets:
        net.destroy()
