"""The 64-bit fixed-point conversion of the fp32 table gradient, on the host:
the function is taken from the kernel's source and compiled with g++."""
import ctypes
import re
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

SRC = Path(__file__).resolve().parents[1] / "paper_2609_34420_amd" / "csrc" / "bwd_f32.hip"


@pytest.fixture(scope="module")
def fixed64(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    m = re.search(r"__device__ __forceinline__ (unsigned long long fixed64\(float xs\) \{.*?\n\})", SRC.read_text(),
                  re.S)
    d = tmp_path_factory.mktemp("fixed")
    (d / "f.cpp").write_text('#include <cmath>\n#include <cstdint>\nextern "C" ' + m.group(1) + "\n")
    subprocess.run([cxx, "-O1", "-ffp-contract=off", "-shared", "-fPIC", str(d / "f.cpp"), "-o", str(d / "f.so")],
                   check=True)
    fn = ctypes.CDLL(str(d / "f.so")).fixed64
    fn.argtypes, fn.restype = [ctypes.c_float], ctypes.c_longlong
    return fn


@pytest.mark.parametrize("sign", [1, -1])
def test_fixed64_rounds_to_nearest(fixed64, sign):
    """Small values of both signs, and 24-bit values of every size up to 2^61:
    the nearest integer, and the value itself where that is one. (A rest of
    exactly 2^31 saturates on the GPU, one unit short; C leaves it open.)"""
    g = np.random.default_rng(0)
    xs = [0.0, 1e-20, 0.25, 0.499, 0.501, 0.75, 1, 1.5, 2, 2.5, 100, 255, 256, 1000, 2 ** 24 - 1, 2.0 ** 31 + 2 ** 8,
          2.0 ** 32 - 2 ** 8, 2.0 ** 32, 2.0 ** 32 + 2 ** 9, 2.0 ** 53, 2.0 ** 61]
    xs += [float(m) * 2.0 ** e for e in range(-30, 38) for m in g.integers(1, 2 ** 24, 40)]
    for x in xs:
        x = sign * float(np.float32(x))
        if abs(x) % 2.0 ** 32 == 2.0 ** 31:
            continue
        got = fixed64(x)
        assert abs(got - int(x) - (x - int(x))) <= 0.5, (x, got)


def test_f32_histogram_range():
    """A lane adds terms below 2^53 times its P, and none once those sum to
    more than 1.5; 512 lanes at most share a sum."""
    text = SRC.read_text()
    lim, psum = re.search(r"lim = 0x1p(\d+)f / sF", text), re.search(r"row_wild = !\(psum <= ([\d.]+)f\)", text)
    assert float(psum.group(1)) * 2 ** int(lim.group(1)) * 512 < 2 ** 63
