"""The kernels' GELU formula (coefficients read from its source), evaluated in fp32 on the
host, against 64 bits.

Bound, relative to the tail |x| Q(|x|): the fit's error (3e-8); eight Horner steps of one
rounding (u = 2^-24) at a condition of at most 2.4 (sum |c_i| over P(1)), 19 u; t with two
roundings at a sensitivity below 4, 8 u; three products, 3 u; s^2 = z^2 log2(e) / 2 with
three roundings in the exponent, 1.5 z^2 u.  The last sum rounds to u of the result.
"""
import pathlib
import re

import numpy as np

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
