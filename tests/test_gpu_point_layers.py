"""1x1 layers on pixels of one or two 16-byte units against the oracle: on maps of more than 131072 positions the
kernel in which a thread owns one unit of output channels, on smaller ones the kernel for short filter rows."""
import numpy as np
import pytest

import oracle
import paper_1704_04313_amd as cb
from workloads.networks import conv, make_weights, pool

from gpu_util import compare_sequence, to_dev

pytestmark = pytest.mark.gpu


def _frames(C, H, W, n, seed):
    """Small integers with a moving block, so that sums are exact and all lists can be compared."""
    r = np.random.default_rng(seed)
    bg = r.integers(0, 4, (C, H, W)).astype(np.float32)
    out = []
    for t in range(n):
        f = bg.copy()
        f[:, t:t + 5, 2 * t:2 * t + 7] = r.integers(0, 4, (C, 1, 1))
        out.append(f)
    return out


# channels of one and two units with and without padding, one to sixteen units of output, ragged positions; maps
# below and above what is ranked in the kernel, the latter also stored without padding channels (from 2^18 on)
@pytest.mark.parametrize("cin,cout,h,w,bf16", [
    (1, 3, 9, 11, False), (3, 8, 37, 41, False), (4, 16, 64, 65, False), (5, 32, 33, 29, False), (8, 64, 31, 50, False),
    (3, 8, 37, 41, True), (8, 64, 40, 33, True), (3, 20, 19, 23, False),
    (3, 8, 367, 361, False), (4, 16, 363, 365, False), (5, 32, 367, 361, False), (8, 16, 362, 363, False), (3, 64, 367, 361, False),
    (8, 64, 367, 361, False), (8, 64, 725, 727, False), (3, 8, 367, 361, True), (8, 64, 363, 365, True), (5, 16, 515, 513, True),
    (1, 8, 513, 515, False), (2, 3, 513, 515, False), (3, 8, 515, 513, False), (3, 64, 513, 517, False), (5, 8, 515, 513, False),
    (6, 32, 513, 515, False), (7, 16, 515, 517, False), (7, 64, 729, 727, False)])
def test_listed_positions(cin, cout, h, w, bf16):
    L = conv(cin, cout, 1)
    frames = [np.random.default_rng(5).random((cin, h, w), dtype=np.float32)]
    for rows, cols in ((h // 3, w // 2), (h // 2, w - 3), (3, 5)):
        f = frames[-1].copy()
        f[:, 2:2 + rows, 3:3 + cols] += np.float32(0.25 * len(frames))
        frames.append(f)
    compare_sequence([L], make_weights([L], cin), frames, 0.02, bf16=bf16, lists_every_frame=True)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("h,w", [(26, 38), (368, 362), (516, 514)])
def test_detection_of_the_layer_behind_bit_exact(bf16, dense, h, w):
    layers = [conv(3, 8, 1), conv(8, 16, 1), pool(), conv(16, 4, 3, relu=False)]
    r = np.random.default_rng(9)
    params = [None if L.kind != "conv" else (r.integers(-1, 2, (L.cout, L.cin, L.kh, L.kw)).astype(np.float32),
                                             r.integers(-2, 3, L.cout).astype(np.float32)) for L in layers]
    net = cb.CBInfer(layers, params, (3, h, w), 0.5, lists_every_frame=True, dtype=cb.BF16 if bf16 else cb.F32)
    orc = oracle.OracleCBNet(layers, params, 0.5, bf16=bf16)
    net.set_mode(dense)
    for t, f in enumerate(_frames(3, h, w, 4, 3)):
        want = orc.process_frame(f) if not dense else oracle.dense_forward(layers, params, f, bf16=bf16)[-1]
        np.testing.assert_array_equal(net.process_frame(to_dev(f)).cpu().numpy()[0], want, err_msg="frame %d" % t)
        for l in (0, 1, 3) if not dense else ():
            np.testing.assert_array_equal(net.read_list(l, cb.LIST_CHANGED), orc.trace[l]["C"], err_msg="layer %d frame %d" % (l, t))
            np.testing.assert_array_equal(net.read_list(l, cb.LIST_UPDATE), orc.trace[l]["U"], err_msg="layer %d frame %d" % (l, t))
    net.destroy()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("cin,cout,h,w", [(3, 8, 61, 83), (8, 16, 61, 83), (8, 64, 40, 52), (6, 32, 128, 1024)])
def test_same_bits_however_positions_arrive(cin, cout, h, w, bf16):
    """Real-valued data: positions ranked in the kernel, from the list of every frame, and all of them in
    order must give the same sums bit for bit (and with them the same flags for the layer behind)."""
    layers = [conv(cin, cout, 1), conv(cout, 8, 3, relu=False)]
    params = make_weights(layers, cin + cout)
    r = np.random.default_rng(h)
    frames = [r.standard_normal((cin, h, w), dtype=np.float32) for _ in range(3)]  # every position changes
    out = {}
    for name, kw in (("ranked", {}), ("listed", {"lists_every_frame": True}), ("dense", {})):
        net = cb.CBInfer(layers, params, (cin, h, w), 0.0, dtype=cb.BF16 if bf16 else cb.F32, **kw)
        net.set_mode(name == "dense")
        out[name] = []
        for f in frames:
            y = net.process_frame(to_dev(f)).cpu().numpy()
            out[name] += [net.read_map(0, cb.MAP_OUTPUT), y]
        net.destroy()
    for a, b, c in zip(out["ranked"], out["listed"], out["dense"]):
        np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(a, c)


def test_a_list_shorter_than_the_map_costs_its_share():
    """A quarter of the positions of a large map takes no more than what its values and the launch take."""
    L = conv(8, 32, 1)
    us = []
    for part in (1.0, 0.25):
        net = cb.CBInfer([L], make_weights([L], 4), (8, 1024, 1024), 0.02, dtype=cb.BF16)
        a = np.random.default_rng(3).random((8, 1024, 1024), dtype=np.float32)
        b = a.copy()
        b[:, :int(1024 * part)] += np.float32(0.5)
        a, b = to_dev(a), to_dev(b)
        for f in (a, b, a, b):
            net.process_frame(f)
        assert net.layer_counts(0)[1] == int(1024 * part) * 1024
        net.set_profiling(True)
        for f in (a, b) * 5:
            net.process_frame(f)
        ms, n = net.read_profile(0, cb.STEP_NAMES.index("gemm"))
        us.append(1e3 * ms / n)
        net.destroy()
    assert us[1] <= 0.55 * us[0], us  # measured: 33 us and 12; 24 with all workgroups of the map in use
