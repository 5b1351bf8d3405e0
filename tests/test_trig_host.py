"""The FP64 sine and cosine of the leaf-to-root walks, compiled for the host and compared with 64-bit-mantissa values."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include "trig.hpp"
int main() {
  double x, sc[2], k;
  while (std::fread(&x, sizeof x, 1, stdin) == 1) {
    const int i = mc::sin_tab_index(x, k);
    mc::SinTabE t;
    t.v.x = mc::kSinTab[i][0];
    t.v.y = mc::kSinTab[i][1];
    t.lo.x = mc::kSinTab[i][2];
    t.lo.y = mc::kSinTab[i][3];
    mc::sincos_finish(x, k, t, sc[0], sc[1]);
    std::fwrite(sc, sizeof sc, 1, stdout);
  }
}
"""


@pytest.fixture(scope="module")
def sincos(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("trig")
    src, exe = d / "trig_host.hip", d / "trig_host"
    src.write_text(PROGRAM)
    subprocess.check_call([HIPCC, "-O2", "-std=c++17", "--offload-host-only", "-mfma", "-Wno-unused-command-line-argument",
                           "-I", os.path.join(ROOT, "paper_2604_13323_amd", "csrc"), str(src), "-o", str(exe)])

    def run(x):
        r = subprocess.run([str(exe)], input=np.ascontiguousarray(x, np.float64).tobytes(), stdout=subprocess.PIPE, check=True)
        return np.frombuffer(r.stdout, np.float64).reshape(-1, 2).T

    return run


@pytest.mark.parametrize("size", [1.0, 20.0, 1e5, 1e8, 1e9, 1e13])
def test_any_number_of_turns(sincos, size):
    """The index of the table entry is whole for |x| < 2e14 and the reduction keeps 2^-53 of the reduced angle, so the errors
    stay at a few roundings of a result below 1: 4e-16."""
    x = np.random.default_rng(1).uniform(-size, size, 20000)
    s, c = sincos(x)
    xl = x.astype(np.longdouble)
    assert np.abs(s - np.sin(xl)).max() < 4e-16
    assert np.abs(c - np.cos(xl)).max() < 4e-16


@pytest.mark.parametrize("size", [0.5, 3.2, 20.0, 300.0])
def test_as_exact_as_one_rounding(sincos, size):
    """The corrections to the table's entry are below 0.05 and the rest of the entry is added to them, so their roundings
    are 1/16 of the result's: its root mean square error is the rounded value's own within 5%, the largest error below
    0.6 units of the last place of a result in [1/2, 1)."""
    x = np.random.default_rng(2).uniform(-size, size, 200000)
    xl = x.astype(np.longdouble)
    err, own = [], []
    for got, want in zip(sincos(x), (np.sin(xl), np.cos(xl))):
        err.append((got - want).astype(float))
        own.append((want.astype(np.float64) - want).astype(float))
    assert np.sqrt(np.mean(np.square(err))) < 1.05 * np.sqrt(np.mean(np.square(own)))
    assert np.abs(err).max() < 0.6 * 2.0 ** -53
