"""The rate that bench.py holds a layer's multiplication against is that of the instruction it runs on."""
import os
import subprocess

import numpy as np
import pytest

import bench
import paper_1704_04313_amd as cb
from paper_1704_04313_amd import build
from workloads.networks import conv

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("layer,bf16,peak", [
    (conv(3, 16, 7), False, 157.3), (conv(64, 8, 1), False, 157.3), (conv(16, 16, 3), False, 157.3),
    (conv(3, 64, 3), False, 157.3), (conv(3, 64, 7), False, 2500 / 6), (conv(3, 64, 1), False, 157.3), (conv(16, 64, 7), False, 2500 / 6),
    (conv(256, 64, 1), False, 2500 / 6), (conv(256, 16, 1), False, 157.3), (conv(3, 16, 7), True, 2500), (conv(64, 256, 7), True, 2500)])
def test_matrix_peak(layer, bf16, peak):
    assert bench.matrix_peak(layer, bf16) == pytest.approx(peak)


def test_halves_are_held_against_what_the_library_launches(tmp_path):
    """bench.in_halves against the library's own answer, at lists and maps around its limits: rounds of whole tiles and rests of every
    size, ranges cut in parts and evenly, maps too small for the grid, 64 channels with tiles of 128 and 256 positions."""
    cb.load_library()
    exe = str(tmp_path / "halves_rule")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-std=c++17", "-o", exe,
                    os.path.join(HERE, "halves_rule.cpp"), "-x", "none", build.LIB, "-Wl,-rpath," + os.path.dirname(build.LIB)],
                   check=True)
    r = np.random.default_rng(0)
    cases = []
    for cin, cout, k in [(64, 256, 7), (16, 64, 7), (64, 64, 5), (96, 64, 3), (128, 128, 3), (512, 512, 3), (768, 128, 1), (736, 128, 1),
                         (85, 100, 3), (15, 64, 7), (64, 32, 7), (75, 200, 5), (256, 64, 3), (3, 64, 3)]:
        for outputs in [100, 4096, 4800, 8192, 16384, 32768, 57600, 230400, 1 << 19, (1 << 19) + 1, 1536000]:
            lists = [outputs, outputs - 1, 1, 128 * 32, 128 * 64, 128 * 128, 128 * 256, 128 * 256 + 1, 128 * 300, 128 * 380, 128 * 511]
            lists += r.integers(1, outputs + 1, 12).tolist()
            cases += [(cin, cout, k, outputs, n) for n in lists if 1 <= n <= outputs]
    text = "".join("%d %d %d %d %d\n" % c for c in cases)
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.split()
    assert len(out) == len(cases) and 200 < out.count("1") < len(out) - 200
    for (cin, cout, k, outputs, n), answer in zip(cases, out):
        assert bench.in_halves(conv(cin, cout, k), n, outputs) == (answer == "1"), (cin, cout, k, outputs, n)
