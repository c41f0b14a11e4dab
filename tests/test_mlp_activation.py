"""The polynomials of the fused MLP product's activation (csrc/pa_mlp.hip), on
the CPU: their coefficients, read from the source, evaluated in fp32 with fused
multiply-adds against 64 bits, to the errors that the source and pa.h state."""
import math
import os
import re

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2502_02414_amd", "csrc", "pa_mlp.hip")


def _coefficients(name):
    """p's starting value and the addends of its fmaf steps."""
    with open(SRC) as f:
        body = re.search(r"float %s\(float x\) \{(.*?)\n\}" % name, f.read(), re.S).group(1)
    c = [re.search(r"float p = ([-\d.e]+)f;", body).group(1)]
    c += re.findall(r"p = fmaf\(p, z, ([-\d.e]+)f\);", body)
    return np.array(c, np.float32), body


def _fma(a, b, c):
    # (the product of two fp32 values is exact in 64 bits)
    return (a.astype(np.float64) * b.astype(np.float64) + np.float64(c)).astype(np.float32)


def _tail(name, z):
    c, body = _coefficients(name)
    p = np.full_like(z, c[0])
    for k in c[1:]:
        p = _fma(p, z, k)
    return np.exp2(p.astype(np.float64)).astype(np.float32), len(c) - 1, body


def _gelu(x):
    z = np.abs(x)
    q, degree, _ = _tail("gelu_ap", z)
    assert degree == 10
    return _fma(-z, q, np.maximum(x, 0))


def _slope(x):
    z = np.abs(x)
    e, degree, body = _tail("dgelu_ap", z)
    assert degree == 11
    z0 = np.float32(re.search(r"\(z - ([\d.]+)f\)", body).group(1))
    v = ((z - z0) * e).astype(np.float32)
    return np.where(x < 0, -v, np.float32(1) + v)


def _exact(x):
    x = x.astype(np.float64)
    Phi = 0.5 * np.array([math.erfc(-t / math.sqrt(2)) for t in x])
    phi = np.exp(-0.5 * x * x) / math.sqrt(2 * math.pi)
    return x * Phi, Phi + x * phi


def _x(lo, hi, n=20001):
    return np.linspace(lo, hi, n).astype(np.float32)


@pytest.mark.parametrize("lo,hi,bar", [(-1, 0, 7.0e-7), (-3, -1, 3.8e-5), (-5, -3, 2.4e-4),
                                       (-12.9, -5, 1.5e-3)])
def test_gelu_relative_error(lo, hi, bar):
    x = _x(lo, hi)
    x = x[x != 0]
    ref = _exact(x)[0]
    assert np.max(np.abs(_gelu(x) / ref - 1)) <= 1.05 * bar


@pytest.mark.parametrize("lo,hi,bar", [(-4, -3, 2.2e-5), (-6, -4, 5.1e-5), (-13, -6, 2.7e-4)])
def test_slope_relative_error(lo, hi, bar):
    x = _x(lo, hi)
    assert np.max(np.abs(_slope(x) / _exact(x)[1] - 1)) <= 1.05 * bar


def test_absolute_errors():
    x = np.concatenate([_x(-13, 0), _x(1e-3, 13)])
    neg, pos = x[x <= 0], x[x > 0]
    for part in (neg, pos):
        g, s = _exact(part)
        assert np.max(np.abs(_gelu(part) - g) / np.maximum(1, np.abs(g))) <= 1.6e-7
        assert np.max(np.abs(_slope(part) - s)) <= 1.8e-7
