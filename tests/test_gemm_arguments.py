"""The multiplication's host entry refuses arguments whose derived fields (the words that its ranking holds in LDS, the way its
producers address rows) were made for other arguments, as it does for the divisors: nothing may be launched with them."""
import os
import subprocess

import pytest

import paper_1704_04313_amd as cb
from paper_1704_04313_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_stale_derived_fields_are_refused(tmp_path):
    import torch
    if torch.cuda.is_available():
        pytest.skip("the unchanged arguments point to host memory: not for a machine that could launch them")
    cb.load_library()
    exe = str(tmp_path / "gemm_arguments")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-std=c++17", "-o", exe,
                    os.path.join(HERE, "gemm_arguments.cpp"), "-x", "none", build.LIB, "-Wl,-rpath," + os.path.dirname(build.LIB)],
                   check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    answers = {name: int(code) for name, code in (line.split() for line in out.splitlines())}
    invalid = 1  # hipErrorInvalidValue
    assert answers.pop("unchanged") not in (0, invalid)  # no device here
    assert len(answers) == 7 and set(answers.values()) == {invalid}, answers
