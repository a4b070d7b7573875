"""The GELU polynomial of the kernels, evaluated on the CPU in fp32 from the
coefficients of the source file, against the normal tail in float64."""
import os
import re

import numpy as np
from scipy.special import erfc

from paper_2605_01060_amd import build as B


def _coefficients():
    text = open(os.path.join(B.CSRC, "device_common.h")).read()
    body = text[text.index("float gelu_erf(float z)"):]
    body = body[:body.index("return")]
    number = r"(-?\d+\.\d+(?:e-\d+)?)f"
    first = re.search(rf"fmaf\({number}, az, {number}\)", body).groups()
    rest = re.findall(rf"fmaf\(p, az, {number}\)", body)
    assert len(rest) == 6
    return [np.float32(c) for c in (*first, *rest)]


def _poly32(x):
    """Horner steps as fused multiply-adds: one rounding each."""
    wide = np.longdouble
    c = _coefficients()
    p = np.full(x.shape, c[0], np.float32)
    with np.errstate(over="ignore"):  # -inf for huge x, whose power is 0
        for k in c[1:]:
            p = (p.astype(wide) * x.astype(wide) + wide(k)).astype(np.float32)
    return p


def _gelu32(z):
    az = np.abs(z)
    tail = np.exp2(_poly32(az).astype(np.float64)).astype(np.float32)
    wide = np.longdouble
    return (np.maximum(z, 0).astype(wide) - az.astype(wide) * tail.astype(wide)).astype(np.float32)


def test_gelu_error_in_fp32():
    x = np.linspace(0, 30, 600_001).astype(np.float32)
    z = np.concatenate([-x, x])
    ref = 0.5 * z.astype(np.float64) * erfc(-z.astype(np.float64) / np.sqrt(2.0))
    assert np.abs(_gelu32(z) - ref).max() <= 3e-7
    normal = np.random.default_rng(0).standard_normal(400_000).astype(np.float32)
    ref = 0.5 * normal.astype(np.float64) * erfc(-normal.astype(np.float64) / np.sqrt(2.0))
    assert np.sqrt(np.mean((_gelu32(normal) - ref) ** 2)) <= 4.6e-8


def test_gelu_tail_goes_to_zero():
    x = np.concatenate([np.linspace(6, 60, 200_001), np.logspace(2, 38, 1000)]).astype(np.float32)
    p = _poly32(x)
    bound = -27.99 - (x.astype(np.float64) - 6) / 2
    assert np.all(p < bound)
    assert np.all(_gelu32(-x[x > 40]) >= -1e-12)
