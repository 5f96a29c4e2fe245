"""The polynomial cores of the binary64 Exact edge kernel (exact.hip): the
coefficients in the kernel source are the committed fit's, and evaluated in
binary64 as the device does they give atan on |s| <= tan(pi/8) and 2 atanh on
|t| <= 3 - 2 sqrt(2) within one unit in the last place (2.3e-16): half a unit
from the last addition, and the polynomial term's few roundings at under 6%
(atan) and 1% (atanh) of the result."""
import os
import re
import sys

import numpy as np
import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2410_15227_amd", "csrc")
sys.path.insert(0, CSRC)
import fit_cores  # noqa: E402


def coefficients(name, count):
    src = open(os.path.join(CSRC, "exact.hip")).read()
    block = src[src.index(f"double {name} = -0." if name == "A" else f"double {name} = 0."):]
    return [float(v) for v in re.findall(r"(-?\d\.\d+)\)?;", block)[:count]]


@pytest.mark.parametrize("name", ["A", "B"])
def test_binary64_cores(name):
    fit, bound = fit_cores.fit_atan64() if name == "A" else fit_cores.fit_atanh64()
    C = coefficients(name, len(fit))
    assert C == fit and bound < 4e-16
    x = np.linspace(1e-9, fit_cores.TAN_PI_8 if name == "A" else fit_cores.ATANH_T, 100001)
    z = x * x
    p = np.full_like(x, C[0])
    for c in C[1:]:
        p = p * z + c
    got = x + (x * z) * p if name == "A" else 2.0 * x + (x * z) * p
    xl = x.astype(np.longdouble)
    want = np.arctan(xl) if name == "A" else 2 * np.arctanh(xl)
    assert float(np.max(np.abs((got - want) / want))) < 2.3e-16
