"""The run kernel's 10^x (the lambdas of the smoothing's search) against 50
digits. The finalize kernel takes the device library's pow (1.24 units in the last
place), so the run kernel's may be off by no more: half a unit for the last
addition, and an eighth for the two roundings of its second term (below 0.08, of
a result of at least 0.7)."""

import ctypes as C
import os
import shutil
import subprocess
from decimal import Decimal, getcontext

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1202_2355_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None,
                    reason="hipcc not available")
def test_pow10_is_as_close_as_the_library(tmp_path):
    src = tmp_path / "p.hip"
    src.write_text('#include "m2m_pow10.h"\n'
                   'extern "C" double p10(double x) { return m2m::pow10_of(x); }\n')
    so = str(tmp_path / "p.so")
    subprocess.run([HIPCC, "-O3", "-std=c++17", "-shared", "-fPIC", "--offload-host-only", "-x", "hip",
                    "-I", CSRC, "-o", so, str(src)], check=True, capture_output=True)
    f = C.CDLL(so).p10
    f.restype, f.argtypes = C.c_double, [C.c_double]
    getcontext().prec = 50
    rng = np.random.default_rng(1)
    xs = np.concatenate([rng.uniform(-30, 30, 20000), rng.uniform(-0.4, 0.4, 500), rng.uniform(-290, 290, 500),
                         np.arange(-40, 41) * 0.25, [k * np.log10(2.0) * 0.5 for k in range(-40, 41)]])
    worst = 0.0
    for x in map(float, xs):
        ref = Decimal(10) ** Decimal(x)
        err = abs(Decimal(f(x)) - ref)
        ulp = Decimal(float(np.spacing(float(ref))))
        worst = max(worst, float(err / ulp))
    assert worst <= 0.625, worst
    assert f(0.0) == 1.0 and f(1.0) == 10.0 and f(400.0) == np.inf and f(-400.0) == 0.0
