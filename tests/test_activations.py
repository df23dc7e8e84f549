"""The fitted GELUs of the bf16 epilogues against the normal distribution function (CPU: their
coefficients are read from the source and evaluated in fp32 arithmetic, with the exponential
rounded once; the hardware's is good to one unit in the last place)."""
import os
import re

import numpy as np
import pytest

scipy_special = pytest.importorskip("scipy.special")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F = np.float32


def _coefficients(name):
    src = open(os.path.join(ROOT, "paper_2503_08467_amd", "csrc", "common.h"), encoding="utf-8").read()
    body = src.split(f"float {name}(float u) {{", 1)[1].split("\n}", 1)[0]
    c = [body.split("float p = ", 1)[1].split("f;", 1)[0]] + re.findall(r"p = fmaf\(p, a, ([^)]+)f\)", body)
    return [F(v) for v in c]


def _gelu(u, name="act_gelu_fast"):
    a, coefficients = np.abs(u), _coefficients(name)
    p = np.full_like(u, coefficients[0])
    with np.errstate(over="ignore"):
        for c in coefficients[1:]:
            p = (p.astype(np.float64) * a + np.float64(c)).astype(F)  # one rounding, as fmaf
    e = np.exp2(p.astype(np.float64)).astype(F)
    return (np.maximum(u, 0).astype(np.float64) - a.astype(np.float64) * e).astype(F)


def _exact(u):
    u = u.astype(np.float64)
    return 0.5 * u * scipy_special.erfc(-u / np.sqrt(2.0))


def test_gelu_fit_absolute_error():
    u = np.linspace(-13, 13, 520001).astype(F)
    assert len(_coefficients("act_gelu_fast")) == 9
    # Abramowitz & Stegun 7.1.26, which it replaced: 3.3e-7 at most, 5.45e-8 root mean square
    assert np.max(np.abs(_gelu(u) - _exact(u))) <= 2.7e-7
    n = np.random.default_rng(0).standard_normal(400000).astype(F)
    assert np.sqrt(np.mean((_gelu(n) - _exact(n)) ** 2)) <= 4.0e-8


@pytest.mark.parametrize("lo,hi,rel", [(-3, -1, 2e-5), (-4, -3, 2e-4), (-5, -4, 1.3e-3), (-7, -5, 2.7e-3),
                                       (-8, -7, 8.5e-3), (-9, -8, 1.3e-2)])
def test_gelu_fit_negative_tail(lo, hi, rel):
    # bounds no larger than the replaced formula's own errors there (5.2e-5 .. 1.5e-2)
    u = np.linspace(lo, hi, 100001).astype(F)
    x = _exact(u)
    assert np.max(np.abs(_gelu(u) - x) / np.abs(x)) <= rel


def test_gelu_fit_far_out():
    u = np.concatenate([np.geomspace(9, 1e30, 4000), [3e38]]).astype(F)
    assert np.array_equal(_gelu(u), u)
    assert np.max(np.abs(_gelu(-u))) <= 1e-17


def test_gelu_near_is_no_worse_than_erff():
    u = np.linspace(-13, 13, 520001).astype(F)
    n = np.random.default_rng(0).standard_normal(400000).astype(F)
    erf32 = lambda v: (F(0.5) * v) * (F(1) + scipy_special.erf((v * F(0.70710678)).astype(np.float64)).astype(F))  # noqa: E731
    near = lambda v: _gelu(v, "act_gelu_near")  # noqa: E731
    assert len(_coefficients("act_gelu_near")) == 11
    assert np.max(np.abs(near(u) - _exact(u))) <= 2.6e-7 < np.max(np.abs(erf32(u) - _exact(u)))
    rms = lambda f: np.sqrt(np.mean((f(n) - _exact(n)) ** 2))  # noqa: E731
    assert rms(near) <= 2.2e-8 < rms(erf32)
    t = u[u > -9]
    assert np.max(np.abs(near(t) - _exact(t)) / np.maximum(np.abs(_exact(t)), 1e-30)) <= 4.6e-4
    far = np.concatenate([np.geomspace(9, 1e30, 4000), [3e38]]).astype(F)
    assert np.array_equal(near(far), far) and np.max(np.abs(near(-far))) <= 1e-17
