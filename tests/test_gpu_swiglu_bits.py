"""The SwiGLU epilogue's product (swiglu() in echo_device.h) for every fp32 gate that a product of saturated halves can come to: the bits of
x / (1.0f + expf(-x)) * u wherever the half behind it is not zero, and its distance from 64 bits.

The error's bound: the exponential's argument rounds by 2^-25 (2^-25.5 of the exponential), the exponential itself by one ulp, the sum with 1, the quotient and the
product with u by half of one each: 2.7 ulp of 2^-23."""
import os
import subprocess

import pytest

from paper_2602_02192_amd import build

pytestmark = pytest.mark.gpu


def test_every_gate():
    if not os.path.exists(build.SWEEP):
        build.build_sweep()
    r = subprocess.run([build.SWEEP], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    lines = [[float(v) for v in l.split()] for l in r.stdout.splitlines()]
    assert len(lines) == 5
    for u, tried, halves, floats, rel in lines:
        assert tried > 2.9e9 and halves == 0 and floats == 0 and rel <= 2.7 * 2.0 ** -23, (u, tried, halves, floats, rel)
