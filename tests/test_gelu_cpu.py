"""The kernels' GELU formula (coefficients read from its source), evaluated in fp32 on the
host, against 64 bits.

Bound, relative to the tail |x| Q(|x|): the fit's error (3e-8); eight Horner steps of one
rounding (u = 2^-24) at a condition of at most 2.4 (sum |c_i| over P(1)), 19 u; t with two
roundings at a sensitivity below 4, 8 u; three products, 3 u; s^2 = z^2 log2(e) / 2 with
three roundings in the exponent, 1.5 z^2 u.  The last sum rounds to u of the result.
"""
import ctypes
import pathlib
import re
import subprocess

import numpy as np
import pytest

SRC = pathlib.Path(__file__).parents[1] / "paper_2609_32869_amd" / "csrc" / "wf_common.h"


def test_gelu_formula():
    from scipy.special import erfc
    body = re.search(r"float gelu_erf\(float x\) \{(.*?)\n\}", SRC.read_text(), re.S).group(1)
    c = float(re.search(r"fmaf\(([\d.]+)f, z, 1\.0f\)", body).group(1))
    poly = [float(re.search(r"float p = (\S+?)f;", body).group(1))]
    poly += [float(v) for v in re.findall(r"p = fmaf\(p, t, (\S+?)f\);", body)]
    scale = float(re.search(r"s = z \* ([\d.]+)f;", body).group(1))
    assert len(poly) == 9
    f = np.float32

    def fma(a, b, d):
        return (a.astype(np.float64) * np.float64(b) + np.float64(d)).astype(f)

    x = np.linspace(-8, 8, 100001).astype(f)
    z = np.abs(x)
    t = (f(1) / fma(z, f(c), 1.0)).astype(f)
    p = np.full_like(z, poly[0])
    for k in poly[1:]:
        p = fma(p, t, f(k))
    s = z * f(scale)
    q = (p * t) * np.exp2((-s * s).astype(np.float64)).astype(f)
    got = (np.maximum(x, f(0)).astype(np.float64) - z.astype(np.float64) * q).astype(f)
    x64 = x.astype(np.float64)
    want = 0.5 * x64 * erfc(-x64 / np.sqrt(2))
    eps = 2.0 ** -24
    tail = z * 0.5 * erfc(z.astype(np.float64) / np.sqrt(2))
    bound = tail * (3.1e-8 + (30 + 1.5 * z.astype(np.float64) ** 2) * eps) + eps * np.abs(want) + 1e-30
    err = np.abs(got - want)
    assert (err <= bound).all() and err.max() <= 2.5e-7


@pytest.fixture(scope="module")
def gelu(tmp_path_factory):
    """The header's function, compiled for the host with exact division and exp2."""
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


def test_gelu_limits(gelu):
    inf, big = np.float32(np.inf), np.finfo(np.float32).max
    y = gelu(np.array([inf, big, 1e30, -big, -1e30, -40, 0], np.float32))
    assert y.tolist() == [inf, big, np.float32(1e30), 0, 0, 0, 0]
    assert np.isnan(gelu(np.array([-inf, np.nan], np.float32))).all()
