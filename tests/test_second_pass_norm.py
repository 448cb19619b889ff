"""The norm after the second Gram-Schmidt pass, from the squared norms before it (the device function,
compiled for the host): as accurate as summing the squares of the vector itself down to the
breakdown test, and not a number where that is not one."""
import ctypes
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2401_13926_amd" / "csrc"


@pytest.fixture(scope="module")
def norm(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("norm")
    (d / "hip").mkdir()  # kernels.hpp's only include, not needed here
    (d / "hip" / "hip_runtime.h").write_text("")
    (d / "norm.cpp").write_text('#include <cmath>\n#include <cstdint>\nusing std::sqrt;\n#define __device__\n'
                                '#define __forceinline__ inline\n#include "kernels.hpp"\n'
                                'extern "C" double norm(double ww, double hh) { return kkt::second_pass_norm(ww, hh); }\n')
    subprocess.run([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-I", str(d), "-I", str(CSRC), "-o", str(d / "norm.so"),
                    str(d / "norm.cpp")], check=True)
    f = ctypes.CDLL(str(d / "norm.so")).norm
    f.restype, f.argtypes = ctypes.c_double, [ctypes.c_double, ctypes.c_double]
    return f


@pytest.mark.parametrize("cols", [1, 5, 30])
@pytest.mark.parametrize("ratio", [1.0, 1e-4, 1e-8, 1e-12, 1e-13, 2e-14])
def test_norm_down_to_the_breakdown_test(norm, cols, ratio):
    """w0 = V c + ratio u with u orthogonal to V: after the first pass w is about ratio ||w0||."""
    n = 2000
    rng = np.random.default_rng(cols)
    q = np.linalg.qr(rng.standard_normal((n, cols + 1)))[0]
    v = np.ascontiguousarray(q[:, :cols])
    c = rng.standard_normal(cols)
    w = v @ (c / np.linalg.norm(c)) + ratio * q[:, cols]
    w = w - v @ (v.T @ w)  # first pass, in double
    h = v.T @ w
    got = norm(float(w @ w), float(h @ h))
    exact = np.linalg.norm((w.astype(np.longdouble) - v.astype(np.longdouble) @ (v.T.astype(np.longdouble) @ w)).astype(float))
    # n + cols rounded terms in the sums, halved by the root; V's columns orthonormal to a few units
    # and h of at most 100 units of ||w0||, that is 5e-15 / 2e-14 of ||w||: its square as cancellation
    assert abs(got - exact) <= (n + 100) * 2.0 ** -53 * exact
    assert got > 1e-14 * np.linalg.norm(v @ c / np.linalg.norm(c))


def test_norm_of_what_is_no_number(norm):
    inf, nan = float("inf"), float("nan")
    assert np.isnan(norm(inf, inf)) and np.isnan(norm(nan, 1.0)) and np.isnan(norm(1.0, nan))
    assert norm(inf, 1.0) == inf and norm(1.0, 1.0 + 2e-16) == 0.0 and norm(1.0, 2.0) == 0.0 and norm(4.0, 0.0) == 2.0
