"""The kernels' GELU (its function compiled for the host from the kernels' header, with exact
division and exp2 in place of the two instructions) against 64 bits.

Bound: Q = E (1 / 2 + s G(s)) with q = erfcx(z / sqrt(2)) / 2 its second factor.  The fit is
within 1e-8 of q, the stored coefficients within u (u = 2^-24) of theirs, and ten fused steps
round once each: 11 u (1 / 2 + sum |c_i| s^(i + 1)); s has three roundings, the reciprocal one
more, each to within 2 u: 5 u sum (i + 1) |c_i| s^(i + 1).  E has 1 u, and y^2 in its
exponent three roundings: 1.5 z^2 u; their product 1 u.  The last sum rounds to u of the result.
"""
import ctypes
import pathlib
import subprocess

import numpy as np
import pytest
from scipy.special import erfc, erfcx

SRC = pathlib.Path(__file__).parents[1] / "paper_2609_32869_amd" / "csrc" / "wf_common.h"
U = 2.0 ** -24


@pytest.fixture(scope="module")
def gelu(tmp_path_factory):
    text = SRC.read_text()
    at = text.index("float gelu_erf(float x)")
    function = text[at:text.index("\n}", at) + 2]
    folder = tmp_path_factory.mktemp("gelu")
    (folder / "gelu.cpp").write_text(
        "#include <cmath>\nusing namespace std;\n"
        "static float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }\n"
        "static float __builtin_amdgcn_exp2f(float x) { return (float)exp2((double)x); }\n"
        f"static {function}\n"
        'extern "C" void run(const float* x, float* y, long n) { for (long i = 0; i < n; ++i) y[i] = gelu_erf(x[i]); }\n')
    # every fma and rounding as written
    subprocess.run(["g++", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-o", folder / "gelu.so", folder / "gelu.cpp"],
                   check=True)
    lib = ctypes.CDLL(str(folder / "gelu.so"))

    def run(x):
        x = np.ascontiguousarray(x, np.float32)
        y = np.empty_like(x)
        lib.run(ctypes.c_void_p(x.ctypes.data), ctypes.c_void_p(y.ctypes.data), ctypes.c_long(x.size))
        return y
    return run


def exact(x):
    x = x.astype(np.float64)
    return 0.5 * x * erfc(-x / np.sqrt(2))


# s = SCALE z / (1 + SCALE z) and G's coefficients, highest power first (for the bound alone)
SCALE = 0.335
G = [0.0277183522, -0.0968085453, 0.0924139991, 0.00293521956, 0.0606820174, -0.160599366, -0.272231847, 1.03676665,
     -1.19087183]


def test_gelu_formula(gelu):
    x = np.linspace(-8, 8, 100001).astype(np.float32)
    z = np.abs(x).astype(np.float64)
    s = SCALE * z / (1 + SCALE * z)
    size = [abs(k) * s ** (9 - i) for i, k in enumerate(G)]  # |c_i| s^(i + 1), highest first
    slope = [(9 - i) * v for i, v in enumerate(size)]
    q, E = erfcx(z / np.sqrt(2)) / 2, np.exp(-z * z / 2)
    bound = z * E * (1e-8 * q + U * (11 * (0.5 + sum(size)) + 5 * sum(slope)) + U * q * (2 + 1.5 * z * z))
    want = exact(x)
    err = np.abs(gelu(x) - want)
    assert (err <= bound + U * np.abs(want) + 1e-30).all() and err.max() <= 2.5e-7


def test_gelu_keeps_small_values(gelu):
    """Relative error near zero, where 0.5 x (1 + erf(x / sqrt(2))) in fp32 is within 2 u."""
    x = np.linspace(-0.2, 0.2, 100001).astype(np.float32)
    x = x[x != 0]
    want = exact(x)
    err = np.abs(gelu(x) - want) / np.abs(want)
    assert err.max() <= 2.7 * U and np.sqrt((err ** 2).mean()) <= 0.7 * U


def test_gelu_limits(gelu):
    inf, big = np.float32(np.inf), np.finfo(np.float32).max
    y = gelu(np.array([inf, big, 1e30, -big, -1e30, -40, 0], np.float32))
    assert y.tolist() == [inf, big, np.float32(1e30), 0, 0, 0, 0]
    assert np.isnan(gelu(np.array([-inf, np.nan], np.float32))).all()
