"""cos and sin of the rotary embedding's angles, from the library's own source built for the host, against extended
precision over angles up to 2^31: the fp32 results are correctly rounded but for ties."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2604_16498_amd import build

SHIM = """
#define __host__
#define __device__
#include "%s"
extern "C" void cos_sin_all(const double* a, float* c, float* s, long n) {
  for (long i = 0; i < n; ++i) forge::cos_sin(a[i], c[i], s[i]);
}
"""


def test_cos_sin_over_all_positions(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision to compare with")
    src, lib = tmp_path / "shim.cpp", tmp_path / "shim.so"
    src.write_text(SHIM % os.path.join(build.CSRC, "angles.hpp"))
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-ffp-contract=off", str(src), "-o", str(lib)], check=True)
    rng = np.random.default_rng(7)
    n = 400000
    half_pi = np.arccos(np.longdouble(0.0))
    k = np.concatenate([np.arange(2000), rng.integers(0, int(2**31 / 1.6), n // 2)])
    angles = np.concatenate([
        rng.uniform(0, 2**31, n), np.exp2(rng.uniform(-40, 31, n)), rng.integers(0, 2**31, n).astype(np.float64),
        np.asarray(k * half_pi, dtype=np.float64),                              # next to the quadrants' ends ...
        np.asarray((k + np.longdouble(0.5)) * half_pi, dtype=np.float64),       # ... and middles
        np.nextafter(np.asarray(k * half_pi, dtype=np.float64), 0.0),
        [0.0, np.nextafter(2.0**31, 0.0)],
    ])
    angles = np.ascontiguousarray(angles[(angles >= 0) & (angles < 2.0**31)])
    c, s = np.empty(angles.size, np.float32), np.empty(angles.size, np.float32)
    ptr = lambda a: a.ctypes.data_as(C.c_void_p)
    C.CDLL(str(lib)).cos_sin_all(ptr(angles), ptr(c), ptr(s), C.c_long(angles.size))
    for got, fn in ((c, np.cos), (s, np.sin)):
        exact = fn(angles.astype(np.longdouble))
        # half a unit of fp32, and 4e-16 for the fp64 series and its reduction (2e-16 measured)
        bound = 0.5 * np.spacing(np.abs(exact).astype(np.float32)).astype(np.longdouble) + 4e-16 * np.abs(exact) + 1e-24
        worst = np.max(np.abs(got.astype(np.longdouble) - exact) / bound)
        assert worst <= 1.0, worst
